// Spherical harmonic transform of fields on an equiangular grid (Sec. III.A.1,
// "Modeling in the Spherical Harmonic Domain"; the precomputation of
// Sec. III.A.2) and its inverse, used to turn emulated coefficient vectors
// back into fields (Sec. III.B), batched over time steps, and the C ABI of the
// transform object (include/mpchol.h).
//
// The paper's route: G_m(theta_j) by FFT along longitude; G_m extended to
// colatitudes in (pi, 2 pi) with G_m(2 pi - theta) = (-1)^m G_m(theta) and an
// FFT along the extended colatitude gives K_{m,m'}; the coefficients follow
// from K through Wigner-d functions at pi/2, precomputed by a three-term
// recursion.  Every step after the longitude FFT is linear in G_m and the
// same for all time steps, so on the GPU the steps are composed once, at
// set-up, into one real table per order m (Sec. III.A.2 precomputes the
// Wigner-d part; here the colatitude DFT and both sums are precomputed too):
//   * the two sums (over m' with I(m' + m'') and over m'' with S_{l,m,m''})
//     fold into a table over m' >= 0, using K_{m,-m'} = (-1)^m K_{m,m'}, the
//     cancellation of the q = +-1 terms of I(q) under that symmetry, and
//     d^l_{m'',0}(pi/2) = 0 for l + m'' odd (degree l meets only m' = l mod 2);
//   * the colatitude DFT of the extended G_m, written out with that symmetry,
//     weighs G_m(theta_j) by 2 cos(m' theta_j) (m even) or -2i sin(m' theta_j)
//     (m odd, pole samples zero); composed with the folded table it gives
//     z_{l,m} = i^{-m-(m mod 2)} sum_j a_{l,j} G_m(theta_j) with a real;
//   * a_{l, pi - theta} = (-1)^{l+m} a_{l,theta}, so only the northern half of
//     the colatitudes is kept: rows j and N_theta - 1 - j are transformed
//     together (two real rows per complex FFT) and enter as
//     G_j + G_{N-1-j} (l + m even) or G_j - G_{N-1-j} (l + m odd).
// Per order m and degree parity p the forward transform is then one real FP64
// MFMA GEMM over all time steps of a batch (columns 2t and 2t + 1 hold the
// real and imaginary parts), and the inverse the mirror image with the table
// 2 pi Y_lm(theta_j, 0) (up to the sign i^{m - (m mod 2)}), composed the same
// way from the paper's K_{m,m'} = 2 pi i^-m sum_l c_l d^l_{m',0} d^l_{m',m} z_{l,m}
// and G_m(theta) = sum_m' K_{m,m'} e^{i m' theta}.  GEMM work per time step
// stays about L^3 flops; the colatitude FFT leaves the per-field path.
// Readings (the grid, the 1/2pi of the longitude synthesis, the poles, the
// real layout of the coefficient vector) are stated with the declarations in
// mpchol.h.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <type_traits>
#include <utility>
#include <vector>

#include "../../include/mpchol.h"
#include "common.h"
#include "gemm_core.h"

namespace mpc {
namespace sht {

constexpr int MAXP = 16;   // passes of a plan
constexpr int MAXN = 4096; // longest transform
constexpr int MAXL = 1024; // band limit (2^-l of the edge value stays a normal double)

struct Plan {
    int n, np;
    int r[MAXP];
};

// GEMM block: 64 rows by 64 columns, K slices of 16, four waves (three workgroups
// share a compute unit; with 128 columns two do: L = 360, 512 fields 0.72 against
// 0.68 ms, L = 720, 64 fields 0.64 against 0.60).  Up to SMALL_T fields (two
// columns each) take blocks of 16 columns, which move and multiply a quarter of it.
constexpr int GBM = 64, GBN = 64, GBK = 16, GNT = 256;
constexpr int SMALL_T = 8;

__device__ inline double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ inline double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ inline double2 cmul(double2 a, double2 b) { return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x); }
__device__ inline double2 cscale(double2 a, double s) { return make_double2(a.x * s, a.y * s); }
// multiply by i^e, e in 0..3
__device__ inline double2 ipow(double2 a, int e)
{
    switch (e & 3) {
    case 1: return make_double2(-a.y, a.x);
    case 2: return make_double2(-a.x, -a.y);
    case 3: return make_double2(a.y, -a.x);
    default: return a;
    }
}

// cos and sin of 2 pi k / R
template <int R> struct Root;
template <> struct Root<6> {
    static constexpr double c[6] = {1.0, 0.5, -0.5, -1.0, -0.5, 0.5};
    static constexpr double s[6] = {0.0, 0.8660254037844386, 0.8660254037844386, 0.0, -0.8660254037844386, -0.8660254037844386};
};
template <> struct Root<8> {
    static constexpr double c[8] = {1.0, 0.7071067811865476, 0.0, -0.7071067811865476, -1.0, -0.7071067811865476, 0.0, 0.7071067811865476};
    static constexpr double s[8] = {0.0, 0.7071067811865476, 1.0, 0.7071067811865476, 0.0, -0.7071067811865476, -1.0, -0.7071067811865476};
};
template <> struct Root<9> {
    static constexpr double c[9] = {1.0, 0.766044443118978, 0.17364817766693036, -0.5, -0.9396926207859084, -0.9396926207859084, -0.5, 0.17364817766693036, 0.766044443118978};
    static constexpr double s[9] = {0.0, 0.6427876096865394, 0.984807753012208, 0.8660254037844386, 0.3420201433256687, -0.3420201433256687, -0.8660254037844386, -0.984807753012208, -0.6427876096865394};
};
template <> struct Root<10> {
    static constexpr double c[10] = {1.0, 0.8090169943749475, 0.30901699437494745, -0.30901699437494745, -0.8090169943749475, -1.0, -0.8090169943749475, -0.30901699437494745, 0.30901699437494745, 0.8090169943749475};
    static constexpr double s[10] = {0.0, 0.5877852522924731, 0.9510565162951535, 0.9510565162951535, 0.5877852522924731, 0.0, -0.5877852522924731, -0.9510565162951535, -0.9510565162951535, -0.5877852522924731};
};
template <> struct Root<12> {
    static constexpr double c[12] = {1.0, 0.8660254037844386, 0.5, 0.0, -0.5, -0.8660254037844386, -1.0, -0.8660254037844386, -0.5, 0.0, 0.5, 0.8660254037844386};
    static constexpr double s[12] = {0.0, 0.5, 0.8660254037844386, 1.0, 0.8660254037844386, 0.5, 0.0, -0.5, -0.8660254037844386, -1.0, -0.8660254037844386, -0.5};
};

// R-point DFT in place in registers: V[q] = sum_r v[r] e^{-2 pi i q r / R}.
// Composite R = R1 R2: R2 transforms of length R1, the roots of R, R1 of length R2.
template <int R> __device__ inline void dft(double2 (&v)[R]);
template <int R1, int R2> __device__ inline void dft_composite(double2 (&v)[R1 * R2])
{
    constexpr int R = R1 * R2;
    double2 y[R2][R1];
    static_for<0, R2>([&](auto N2) {
        constexpr int n2 = N2;
#pragma unroll
        for (int n1 = 0; n1 < R1; ++n1) y[n2][n1] = v[R2 * n1 + n2];
        dft<R1>(y[n2]);
        static_for<1, R1>([&](auto K1) {
            constexpr int e = n2 * K1;
            if constexpr (e > 0) y[n2][K1] = cmul(y[n2][K1], make_double2(Root<R>::c[e], -Root<R>::s[e]));
        });
    });
#pragma unroll
    for (int k1 = 0; k1 < R1; ++k1) {
        double2 z[R2];
#pragma unroll
        for (int n2 = 0; n2 < R2; ++n2) z[n2] = y[n2][k1];
        dft<R2>(z);
#pragma unroll
        for (int k2 = 0; k2 < R2; ++k2) v[k1 + R1 * k2] = z[k2];
    }
}
template <int R> __device__ inline void dft(double2 (&v)[R])
{
    if constexpr (R == 2) {
        const double2 a = v[0], b = v[1];
        v[0] = cadd(a, b);
        v[1] = csub(a, b);
    } else if constexpr (R == 3) {
        const double2 t = cadd(v[1], v[2]), d = cscale(csub(v[1], v[2]), Root<6>::s[1]);
        const double2 u = make_double2(v[0].x - 0.5 * t.x, v[0].y - 0.5 * t.y);
        v[0] = cadd(v[0], t);
        v[1] = make_double2(u.x + d.y, u.y - d.x);
        v[2] = make_double2(u.x - d.y, u.y + d.x);
    } else if constexpr (R == 4) {
        const double2 s02 = cadd(v[0], v[2]), d02 = csub(v[0], v[2]), s13 = cadd(v[1], v[3]), d13 = csub(v[1], v[3]);
        v[0] = cadd(s02, s13);
        v[2] = csub(s02, s13);
        v[1] = make_double2(d02.x + d13.y, d02.y - d13.x);
        v[3] = make_double2(d02.x - d13.y, d02.y + d13.x);
    } else if constexpr (R == 5) {
        constexpr double c1 = Root<10>::c[2], c2 = Root<10>::c[4], s1 = Root<10>::s[2], s2 = Root<10>::s[4];
        const double2 t1 = cadd(v[1], v[4]), t2 = cadd(v[2], v[3]), t3 = csub(v[1], v[4]), t4 = csub(v[2], v[3]);
        const double2 a1 = make_double2(v[0].x + c1 * t1.x + c2 * t2.x, v[0].y + c1 * t1.y + c2 * t2.y);
        const double2 a2 = make_double2(v[0].x + c2 * t1.x + c1 * t2.x, v[0].y + c2 * t1.y + c1 * t2.y);
        const double2 b1 = make_double2(s1 * t3.x + s2 * t4.x, s1 * t3.y + s2 * t4.y);
        const double2 b2 = make_double2(s2 * t3.x - s1 * t4.x, s2 * t3.y - s1 * t4.y);
        v[0] = cadd(v[0], cadd(t1, t2));
        v[1] = make_double2(a1.x + b1.y, a1.y - b1.x);
        v[4] = make_double2(a1.x - b1.y, a1.y + b1.x);
        v[2] = make_double2(a2.x + b2.y, a2.y - b2.x);
        v[3] = make_double2(a2.x - b2.y, a2.y + b2.x);
    } else if constexpr (R == 6) dft_composite<2, 3>(v);
    else if constexpr (R == 8) dft_composite<4, 2>(v);
    else if constexpr (R == 9) dft_composite<3, 3>(v);
    else if constexpr (R == 10) dft_composite<2, 5>(v);
    else if constexpr (R == 12) dft_composite<4, 3>(v);
}

// Element i of a sequence in LDS: one place in 17 is skipped, so that the writes
// of a pass, R elements apart, spread over the banks for even R too.
__host__ __device__ inline int skew(int i) { return i + (i >> 4); }
__host__ __device__ inline int seq_len(int n) { return skew(n) + 1; }

// One Stockham pass of radix R over nseq sequences of length n (in place in LDS:
// every butterfly reads its inputs before a barrier and writes its outputs after
// it).  Ns = product of earlier radices; load(s)(i) and store(s)(i, v) take
// and give element i of sequence s, in LDS or in memory.
// butterflies of a pass per thread: one, of the smallest radices two
__host__ __device__ constexpr int butterflies(int R) { return R <= 3 ? 2 : 1; }

template <int R, typename Load, typename Store>
__device__ inline void fft_pass(int nseq, int n, int Ns, const double2 *tw, Load load, Store store)
{
    constexpr int MB = butterflies(R);
    // the length anew in every pass: otherwise the indices of all radices are
    // computed ahead of the loop over the passes, and spilled
    asm volatile("" : "+s"(n));
    const int nb = n / R;
    double2 v[MB][R];
#pragma unroll
    for (int i = 0; i < MB; ++i) {
        const int idx = threadIdx.x + i * blockDim.x, s = idx / nb, j = idx - s * nb;
        if (s < nseq) {
            auto from = load(s);
#pragma unroll
            for (int r = 0; r < R; ++r) v[i][r] = from(j + r * nb);
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < MB; ++i) {
        const int idx = threadIdx.x + i * blockDim.x, s = idx / nb, j = idx - s * nb;
        if (s < nseq) {
            const int jn = j / Ns, k = j - jn * Ns;
            if (Ns > 1) {
                const int step = k * (n / (Ns * R));
#pragma unroll
                for (int r = 1; r < R; ++r) v[i][r] = cmul(v[i][r], tw[r * step]);
            }
            if constexpr (R > 1) dft<R>(v[i]);
            auto to = store(s);
#pragma unroll
            for (int q = 0; q < R; ++q) to(jn * Ns * R + k + q * Ns, v[i][q]);
        }
    }
    __syncthreads();
}

template <typename Load, typename Store>
__device__ inline void fft_step(int R, int nseq, int n, int Ns, const double2 *tw, Load load, Store store)
{
    switch (R) {
    case 2: fft_pass<2>(nseq, n, Ns, tw, load, store); break;
    case 3: fft_pass<3>(nseq, n, Ns, tw, load, store); break;
    case 4: fft_pass<4>(nseq, n, Ns, tw, load, store); break;
    case 5: fft_pass<5>(nseq, n, Ns, tw, load, store); break;
    case 6: fft_pass<6>(nseq, n, Ns, tw, load, store); break;
    case 8: fft_pass<8>(nseq, n, Ns, tw, load, store); break;
    case 9: fft_pass<9>(nseq, n, Ns, tw, load, store); break;
    case 10: fft_pass<10>(nseq, n, Ns, tw, load, store); break;
    case 12: fft_pass<12>(nseq, n, Ns, tw, load, store); break;
    default: fft_pass<1>(nseq, n, Ns, tw, load, store); break;
    }
}

constexpr int MAXSEQ = 8;  // sequences of an FFT workgroup

// The two rows of a sequence and its place in the blocks of the contraction.
struct Seq {
    int64_t z0, z1;  // first elements of rows j' and N_theta - 1 - j' of the field (equal at the equator)
    int64_t o;       // row j', column 2t of a block; < 0: no such sequence (z0 and z1 then the first row)
};
__device__ inline Seq sequence(int64_t g, int64_t nsq, int T, int ntheta, int n, int64_t ld)
{
    Seq q{0, 0, -1};
    if (g < nsq) {
        const int jp = (int)(g / T), t = (int)(g - (int64_t)jp * T), js = ntheta - 1 - jp;
        q.z0 = ((int64_t)t * ntheta + jp) * n;
        q.z1 = ((int64_t)t * ntheta + js) * n;
        q.o = jp * ld + 2 * t;
    }
    return q;
}

// ------------------------------------------------------------------ longitude
__host__ __device__ inline int lstart(int m, int p) { return ((m & 1) == p) ? m : m + 1; }

// Forward: sequence g = j' T + t (j' < H = ceil(N_theta / 2)) packs rows j' and
// N_theta - 1 - j' of field t (the equator of an odd grid twice, and only its
// first spectrum used); with A, B their spectra times 2 pi / N_phi, block (m, q) of Gb gets
// row j', columns 2t, 2t + 1: A + B (q = 0) and A - B (q = 1), m = 0..L-1.
// Bound by LDS traffic more than by its bytes: the first pass reads the fields
// themselves, radices up to 12 leave three passes for N_phi = 720, and their
// roots are constants (five passes with looked-up roots before: L = 360, 512
// fields 1.03 -> 0.57 ms, 3.7 TB/s).  Workgroups that fill the same lines share an
// XCD.
template <int MAXT>
__global__ __launch_bounds__(MAXT) __attribute__((amdgpu_waves_per_eu(MAXT == 512 ? 3 : 4))) void phi_forward_kernel(const double *__restrict__ Z, int T, int ntheta, int L, Plan P,
                                                          const double2 *__restrict__ twg, double *Gb, int64_t blk,
                                                          int64_t ld, int nseq)
{
    extern __shared__ __align__(16) char smem_raw[];
    __shared__ Seq seq[MAXSEQ];
    const int n = P.n, sl = seq_len(n);
    double2 *tws = (double2 *)smem_raw;
    double2 *buf = tws + n;
    const int64_t g0 = xcd_remap(blockIdx.x, gridDim.x) * nseq;
    if (threadIdx.x < nseq)
        seq[threadIdx.x] = sequence(g0 + threadIdx.x, (int64_t)((ntheta + 1) / 2) * T, T, ntheta, n, ld);
    for (int i = threadIdx.x; i < n; i += blockDim.x) tws[i] = twg[i];
    __syncthreads();
    int Ns = 1;
    for (int p = 0; p < P.np; ++p) {
        auto store = [&](int s) {
            return [b = buf + s * sl](int i, double2 v) { b[skew(i)] = v; };
        };
        if (p == 0)
            fft_step(P.r[0], nseq, n, 1, tws,
                     [&](int s) {
                         return [z0 = Z + seq[s].z0, z1 = Z + seq[s].z1](int i) { return make_double2(z0[i], z1[i]); };
                     },
                     store);
        else
            fft_step(P.r[p], nseq, n, Ns, tws,
                     [&](int s) { return [b = buf + s * sl](int i) { return b[skew(i)]; }; }, store);
        Ns *= P.r[p];
    }
    const double sc = M_PI / n;  // (2 pi / n) / 2 of the two-row separation
    for (int idx = threadIdx.x; idx < nseq * L; idx += blockDim.x) {
        const int m = idx / nseq, s = idx - m * nseq;
        const Seq &q = seq[s];
        if (q.o < 0) continue;
        const double2 X = buf[s * sl + skew(m)], Y = buf[s * sl + skew(m ? n - m : 0)];
        // A = (X + conj Y) / 2, B = (X - conj Y) / 2i, both times 2 pi / n
        const double2 a = make_double2(sc * (X.x + Y.x), sc * (X.y - Y.y));
        const double2 b = make_double2(sc * (X.y + Y.y), -sc * (X.x - Y.x));
        double2 gs = cadd(a, b), ga = csub(a, b);
        if (q.z1 == q.z0) {  // the equator: its row alone
            gs = a;
            ga = make_double2(0.0, 0.0);
        }
        *(double2 *)(Gb + (2 * m) * blk + q.o) = gs;
        *(double2 *)(Gb + (2 * m + 1) * blk + q.o) = ga;
    }
}

// Inverse: for the pair of rows (j', N_theta - 1 - j') of field t, with E and O
// the results of the even (l + m even) and odd blocks of order m,
// G_m = i^{m mod 2 - m} (E + O) on row j' and i^{m mod 2 - m} (E - O) on its
// mirror; Z = (1 / 2 pi) sum_{|m| < L} G_m e^{i m phi}, G_{-m} = conj(G_m), both
// rows from one inverse FFT (their spectra are Hermitian): the forward transform
// with real and imaginary parts exchanged on the way in and out.  The last pass
// writes the fields (L = 720, 64 fields: 0.72 -> 0.43 ms).
template <int MAXT>
__global__ __launch_bounds__(MAXT) __attribute__((amdgpu_waves_per_eu(MAXT == 512 ? 3 : 4))) void phi_inverse_kernel(const double *__restrict__ Ob, int64_t blk, int64_t ld, int T,
                                                          int ntheta, int L, Plan P, const double2 *__restrict__ twg,
                                                          double *__restrict__ Z, int nseq)
{
    extern __shared__ __align__(16) char smem_raw[];
    __shared__ Seq seq[MAXSEQ];
    const int n = P.n, sl = seq_len(n);
    double2 *tws = (double2 *)smem_raw;
    double2 *buf = tws + n;
    const int64_t g0 = xcd_remap(blockIdx.x, gridDim.x) * nseq;
    if (threadIdx.x < nseq)
        seq[threadIdx.x] = sequence(g0 + threadIdx.x, (int64_t)((ntheta + 1) / 2) * T, T, ntheta, n, ld);
    for (int i = threadIdx.x; i < n; i += blockDim.x) tws[i] = twg[i];
    const int gap = n - 2 * L + 1;  // orders L .. n - L
    for (int idx = threadIdx.x; idx < nseq * gap; idx += blockDim.x) {
        const int s = idx / gap;
        buf[s * sl + skew(L + idx - s * gap)] = make_double2(0.0, 0.0);
    }
    __syncthreads();
    const double sc = 1.0 / (2.0 * M_PI);
    for (int idx = threadIdx.x; idx < nseq * L; idx += blockDim.x) {
        const int m = idx / nseq, s = idx - m * nseq;
        const Seq &q = seq[s];
        double2 ga = make_double2(0.0, 0.0), gb = ga;
        if (q.o >= 0) {
            const int p0 = m & 1;  // degree parity of the block with l + m even
            const double2 E = *(const double2 *)(Ob + (2 * m + p0) * blk + q.o);
            const double2 O = *(const double2 *)(Ob + (2 * m + (p0 ^ 1)) * blk + q.o);
            const int e = ((m & 1) - m) & 3;
            ga = cscale(ipow(cadd(E, O), e), sc);
            if (q.z1 != q.z0) gb = cscale(ipow(csub(E, O), e), sc);
        }
        double2 *bs = buf + s * sl;  // parts exchanged
        if (m == 0) {  // G_0 of a real field is real
            bs[0] = make_double2(gb.x, ga.x);
        } else {
            bs[skew(m)] = make_double2(ga.y + gb.x, ga.x - gb.y);       // ga + i gb
            bs[skew(n - m)] = make_double2(gb.x - ga.y, ga.x + gb.y);  // conj(ga) + i conj(gb)
        }
    }
    __syncthreads();
    int Ns = 1;
    for (int p = 0; p < P.np; ++p) {
        auto load = [&](int s) { return [b = buf + s * sl](int i) { return b[skew(i)]; }; };
        if (p + 1 < P.np)
            fft_step(P.r[p], nseq, n, Ns, tws, load, [&](int s) {
                return [b = buf + s * sl](int i, double2 v) { b[skew(i)] = v; };
            });
        else
            fft_step(P.r[p], nseq, n, Ns, tws, load, [&](int s) {
                const Seq &q = seq[s];
                return [z0 = Z + q.z0, z1 = Z + q.z1, on = q.o >= 0, two = q.z1 != q.z0](int i, double2 v) {
                    if (on) z0[i] = v.y;
                    if (on && two) z1[i] = v.x;
                };
            });
        Ns *= P.r[p];
    }
}

// ------------------------------------------------------------------ contraction
struct Item {
    int16_t m, p;
    int32_t tm;
};

// Degrees of block (m, p): l = lstart(m, p) + 2 r, r < block_rows.
__host__ __device__ inline int block_rows(int L, int m, int p)
{
    const int l0 = lstart(m, p);
    return l0 < L ? (L - 1 - l0) / 2 + 1 : 0;
}

// acc += A B over K (a multiple of 16), A(r, k) = A[r + k lda] for 64 rows, B(k, c) =
// B[c + k ldb] for BN columns; WM x WN waves, two K slices in flight in registers
// beside the one in LDS.  Only the first `mt` 16-row tiles are multiplied: the rows
// of a block end anywhere (at L = 360 whole 64-row blocks are a third larger than
// the rows, whole 16-row tiles a tenth).
template <int BN, int WM, int WN> struct SG {
    static constexpr int MB = GBM / WM / 16, NB = BN / WN / 16;
    static constexpr int LDA = GBM + 16, LDB = BN + 16;
    static constexpr int CA = GBM * GBK / 2 / GNT, CHB = BN * GBK / 2, CB = (CHB + GNT - 1) / GNT;
    static constexpr size_t SMEM = sizeof(double) * 2 * GBK * (LDA + LDB);
};
template <int BN, int WM, int WN>
__device__ inline void sht_block(const double *__restrict__ A, int64_t lda, const double *__restrict__ B, int64_t ldb,
                                 int K, int mt, double4_t (&acc)[SG<BN, WM, WN>::MB][SG<BN, WM, WN>::NB], double *smem)
{
    typedef SG<BN, WM, WN> S;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave % WM, wn = wave / WM, gi = lane & 15, gg = lane >> 4;
    double *As = smem, *Bs = smem + 2 * GBK * S::LDA;
    struct Regs {
        u32x4 a[S::CA], b[S::CB];
    } r0, r1;
    const int nk = K / GBK;
    auto gload = [&](int kt, Regs &r) {
#pragma unroll
        for (int c = 0; c < S::CA; ++c) {
            const int ch = tid + GNT * c;
            r.a[c] = *(const u32x4 *)(A + 2 * (ch % (GBM / 2)) + (int64_t)(kt * GBK + ch / (GBM / 2)) * lda);
        }
#pragma unroll
        for (int c = 0; c < S::CB; ++c) {
            const int ch = tid + GNT * c;
            if (S::CHB % GNT == 0 || ch < S::CHB)
                r.b[c] = *(const u32x4 *)(B + 2 * (ch % (BN / 2)) + (int64_t)(kt * GBK + ch / (BN / 2)) * ldb);
        }
    };
    auto sstore = [&](int buf, const Regs &r) {
#pragma unroll
        for (int c = 0; c < S::CA; ++c) {
            const int ch = tid + GNT * c;
            *(u32x4 *)(As + (buf * GBK + ch / (GBM / 2)) * S::LDA + 2 * (ch % (GBM / 2))) = r.a[c];
        }
#pragma unroll
        for (int c = 0; c < S::CB; ++c) {
            const int ch = tid + GNT * c;
            if (S::CHB % GNT == 0 || ch < S::CHB)
                *(u32x4 *)(Bs + (buf * GBK + ch / (BN / 2)) * S::LDB + 2 * (ch % (BN / 2))) = r.b[c];
        }
    };
    auto multiply = [&](int cur, auto M) {
        const double *as = As + cur * GBK * S::LDA + wm * S::MB * 16 + gi;
        const double *bs = Bs + cur * GBK * S::LDB + wn * S::NB * 16 + gi;
#pragma unroll
        for (int s = 0; s < GBK / 4; ++s) {
            double fa[M], fb[S::NB];
#pragma unroll
            for (int m = 0; m < M; ++m) fa[m] = as[(s * 4 + gg) * S::LDA + m * 16];
#pragma unroll
            for (int n = 0; n < S::NB; ++n) fb[n] = bs[(s * 4 + gg) * S::LDB + n * 16];
#pragma unroll
            for (int m = 0; m < M; ++m)
#pragma unroll
                for (int n = 0; n < S::NB; ++n)
                    acc[m][n] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[m], fb[n], acc[m][n], 0, 0, 0);
        }
    };
    const int mw = __builtin_amdgcn_readfirstlane(min(S::MB, mt - wm * S::MB));  // this wave's tiles
    auto compute = [&](int cur) {
        if (mw >= S::MB) multiply(cur, std::integral_constant<int, S::MB>{});
        else if (S::MB > 1 && mw == 1) multiply(cur, std::integral_constant<int, 1>{});
        else if (S::MB > 2 && mw == 2) multiply(cur, std::integral_constant<int, (S::MB > 2 ? 2 : 1)>{});
        else if (S::MB > 2 && mw == 3) multiply(cur, std::integral_constant<int, (S::MB > 2 ? 3 : 1)>{});
    };
    gload(0, r0);
    if (nk > 1) gload(1, r1);
    sstore(0, r0);
    __syncthreads();
    for (int kt = 0;; kt += 2) {
        if (kt + 2 < nk) gload(kt + 2, r0);
        compute(0);
        if (kt + 1 >= nk) break;
        sstore(1, r1);
        __syncthreads();
        if (kt + 3 < nk) gload(kt + 3, r1);
        compute(1);
        if (kt + 2 >= nk) break;
        sstore(0, r0);
        __syncthreads();
    }
}

// One 64 x BN block of a contraction; logical blocks run over the column blocks of
// a row block first and stay in order on an XCD, whose L2 then serves the row
// block's table to all of them and their columns to the next row blocks.  Results
// go row-major (columns contiguous) into block (m, p) of C.
template <int BN, int WM, int WN>
__device__ inline void sht_gemm(const double *A, int64_t lda, const double *B, int64_t ldb, int K, int rows, int tm, int tn,
                                double *C, double *smem)
{
    typedef SG<BN, WM, WN> S;
    double4_t acc[S::MB][S::NB];
#pragma unroll
    for (int a = 0; a < S::MB; ++a)
#pragma unroll
        for (int b = 0; b < S::NB; ++b) acc[a][b] = (double4_t){0.0, 0.0, 0.0, 0.0};
    const int mt = (min(GBM, rows - tm * GBM) + 15) / 16;
    sht_block<BN, WM, WN>(A + tm * GBM, lda, B + tn * BN, ldb, K, mt, acc, smem);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = wave % WM, wn = wave / WM, gi = lane & 15, gg = lane >> 4;
#pragma unroll
    for (int a = 0; a < S::MB; ++a)
        if (wm * S::MB + a < mt)
#pragma unroll
            for (int b = 0; b < S::NB; ++b) {
                const int c = tn * BN + (wn * S::NB + b) * 16 + gi;
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    C[(int64_t)(tm * GBM + (wm * S::MB + a) * 16 + acc_row<double>(gg, v)) * ldb + c] = acc[a][b][v];
            }
}

// Forward: C^{m,p} = A^{m,p} Gq, q = (p + m) mod 2, over the northern colatitudes.
template <int BN, int WM, int WN>
__global__ __launch_bounds__(GNT) void gemm_forward_kernel(const double *__restrict__ Af, const int64_t *__restrict__ aoff,
                                                           const int *__restrict__ arows, const double *__restrict__ Gb,
                                                           int64_t gblk, int64_t ldb, int Kp, int L,
                                                           const Item *__restrict__ items, int ntn, double *Cf, int64_t cblk)
{
    extern __shared__ __align__(16) char smem_raw[];
    const int64_t lg = xcd_remap(blockIdx.x, gridDim.x);
    const Item it = items[lg / ntn];
    const int mp2 = 2 * it.m + it.p;
    sht_gemm<BN, WM, WN>(Af + aoff[mp2], arows[mp2], Gb + (2 * it.m + ((it.p + it.m) & 1)) * gblk, ldb, Kp,
                         block_rows(L, it.m, it.p), it.tm, (int)(lg % ntn), Cf + mp2 * cblk, (double *)smem_raw);
}

// Inverse: E/O^{m,p}[j'][c] = V^{m,p} Bz^{m,p}.
template <int BN, int WM, int WN>
__global__ __launch_bounds__(GNT) void gemm_inverse_kernel(const double *__restrict__ V, const int64_t *__restrict__ voff,
                                                           int64_t ldv, const int *__restrict__ kpadz,
                                                           const double *__restrict__ Bz, const int64_t *__restrict__ zoff,
                                                           int64_t ldb, int H, const Item *__restrict__ items, int ntn,
                                                           double *Ob, int64_t oblk)
{
    extern __shared__ __align__(16) char smem_raw[];
    const int64_t lg = xcd_remap(blockIdx.x, gridDim.x);
    const Item it = items[lg / ntn];
    const int mp2 = 2 * it.m + it.p;
    sht_gemm<BN, WM, WN>(V + voff[mp2], ldv, Bz + zoff[mp2], ldb, kpadz[mp2], H, it.tm, (int)(lg % ntn), Ob + mp2 * oblk,
                         (double *)smem_raw);
}

// Degree of pair pr of a chunk starting at degree la, where degree l holds the
// l + 1 pairs (l, 0..l): the largest l with (l (l+1) - la (la+1)) / 2 <= pr.
__device__ inline int pair_degree(int pr, int la)
{
    const double u = 2.0 * pr + (double)la * (la + 1);
    int l = (int)((sqrt(4.0 * u + 1.0) - 1.0) * 0.5);
    while (l * (l + 1) > u) --l;
    while ((l + 1) * (l + 2) <= u) ++l;
    return l;
}

constexpr int TNT = 1024;  // threads of a transpose workgroup

// Transposes between the coefficient vectors f (T x L^2, degree-major) and the
// per-order GEMM blocks (rows r = (l - lstart(m,p)) / 2, columns 2t / 2t + 1),
// through LDS: a workgroup owns TT time steps and a chunk of whole degrees
// [l_a, l_b) (at most CH coefficients), reads one side contiguously and writes
// the other in runs of 2 TT doubles.
//
// Forward: z_{l,m} = i^{-m-(m mod 2)} (C[r][2t] + i C[r][2t + 1]); f gets z_{l,0}
// and sqrt(2) Re / Im z_{l,m} at l^2 + l +- m.
__global__ __launch_bounds__(TNT) void unpack_forward_kernel(const double *__restrict__ Cf, int64_t cblk, int64_t ldb,
                                      const int *__restrict__ chunk_l, int T, int L, int TT, int CH,
                                      double *__restrict__ f)
{
    extern __shared__ __align__(16) char smem_raw[];
    double *buf = (double *)smem_raw;  // [TT][CH], raw (a at l^2+l+m, b at l^2+l-m)
    const int la = chunk_l[blockIdx.x], lb = chunk_l[blockIdx.x + 1];
    const int i0 = la * la, ni = lb * lb - i0;
    const int t0 = blockIdx.y * TT;
    const int tt = min(TT, T - t0);
    // gather: one (l, m >= 0) pair and 2 tt columns per 2 tt threads; a thread
    // keeps its column and steps through the pairs
    const int npair = (lb * (lb + 1) - la * (la + 1)) / 2;  // sum over l of (l + 1)
    const int dp = TNT / (2 * tt);
    if ((int)threadIdx.x < dp * 2 * tt) {
        const int pr0 = threadIdx.x / (2 * tt), col = threadIdx.x - pr0 * 2 * tt, part = col & 1;
        const double *src = Cf + 2 * t0 + col;
        double *dst = buf + (col / 2) * CH - i0;
        int l = pair_degree(pr0, la), m = pr0 - (l * (l + 1) - la * (la + 1)) / 2;
        for (int pr = pr0; pr < npair; pr += dp) {
            const int p = l & 1, r = (l - lstart(m, p)) >> 1;
            const double v = src[(2 * m + p) * cblk + (int64_t)r * ldb];
            if (m > 0 || part == 0) dst[l * l + l + (part ? -m : m)] = v;
            m += dp;
            while (m > l) m -= ++l;
        }
    }
    __syncthreads();
    for (int idx = threadIdx.x; idx < ni; idx += TNT) {
        const int gi_ = idx + i0;
        int l = (int)sqrt((double)gi_);
        while (l * l > gi_) --l;
        while ((l + 1) * (l + 1) <= gi_) ++l;
        const int ms = gi_ - l * l - l, m = ms < 0 ? -ms : ms;
        // z = i^-rot (a + i b), a at +m, b at -m; sqrt(2) of its real (ms > 0) or imaginary part
        const int rot = (m + (m & 1)) & 3, k = ms > 0 ? rot : (rot + 1) & 3;  // Re: a, b, -a, -b; Im: b, -a, -b, a
        const int from = m == 0 ? idx : (k & 1 ? l * l + l - m : l * l + l + m) - i0;
        const double f0 = m == 0 ? 1.0 : (k & 2 ? -M_SQRT2 : M_SQRT2);
        double *dst = f + (int64_t)t0 * L * L + gi_;
        for (int ts = 0; ts < tt; ++ts) dst[(int64_t)ts * L * L] = f0 * buf[ts * CH + from];
    }
}

// Inverse operand Bz^{m,p}[r][2t] = Re z_{l,m}, [r][2t + 1] = Im z_{l,m} for
// l = lstart + 2r, from f through LDS (same tiling as the forward unpack).
__global__ __launch_bounds__(TNT) void pack_inverse_kernel(const double *__restrict__ f, const int *__restrict__ chunk_l, int T, int L,
                                    int TT, int CH, double *Bz, const int64_t *__restrict__ zoff, int64_t ldb)
{
    extern __shared__ __align__(16) char smem_raw[];
    double *buf = (double *)smem_raw;  // [TT][CH]
    const int la = chunk_l[blockIdx.x], lb = chunk_l[blockIdx.x + 1];
    const int i0 = la * la, ni = lb * lb - i0;
    const int t0 = blockIdx.y * TT;
    const int tt = min(TT, T - t0);
    for (int idx = threadIdx.x; idx < ni; idx += TNT)
        for (int ts = 0; ts < tt; ++ts) buf[ts * CH + idx] = f[(int64_t)(t0 + ts) * L * L + i0 + idx];
    __syncthreads();
    const int npair = (lb * (lb + 1) - la * (la + 1)) / 2;
    const int dp = TNT / (2 * tt);
    if ((int)threadIdx.x < dp * 2 * tt) {
        const int pr0 = threadIdx.x / (2 * tt), col = threadIdx.x - pr0 * 2 * tt, part = col & 1;
        const double *src = buf + (col / 2) * CH - i0;
        double *dst = Bz + 2 * t0 + col;
        int l = pair_degree(pr0, la), m = pr0 - (l * (l + 1) - la * (la + 1)) / 2;
        for (int pr = pr0; pr < npair; pr += dp) {
            const int p = l & 1, r = (l - lstart(m, p)) >> 1;
            double v;
            if (m == 0) v = part ? 0.0 : src[l * l + l];
            else v = src[l * l + l + (part ? -m : m)] * M_SQRT1_2;
            dst[zoff[2 * m + p] + (int64_t)r * ldb] = v;
            m += dp;
            while (m > l) m -= ++l;
        }
    }
}

// ------------------------------------------------------------------ tables
__host__ __device__ inline int64_t wig_off(int l) { return (int64_t)l * (l + 1) * (2 * l + 1) / 6; }

// D[wig_off(l) + k (l+1) + m] = d^l_{k,m}(pi/2) for 0 <= k, m <= l < L: edge value
// d^l_{l,m} = (-1)^(l-m) 2^-l sqrt(C(2l, l+m)) (from m = l down by the ratio
// sqrt((l+m+1)/(l-m))), then the recursion in the first index
// sqrt((l+k)(l-k+1)) d_{k-1,m} = 2m d_{k,m} - sqrt((l-k)(l+k+1)) d_{k+1,m}, k = l..1.
__global__ void wigner_kernel(int L, double *D)
{
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= (int64_t)L * (L + 1) / 2) return;
    int l = (int)((sqrt(8.0 * (double)g + 1.0) - 1.0) * 0.5);
    while ((int64_t)l * (l + 1) / 2 > g) --l;
    while ((int64_t)(l + 1) * (l + 2) / 2 <= g) ++l;
    const int m = (int)(g - (int64_t)l * (l + 1) / 2);
    double e = ldexp(1.0, -l);
    for (int mm = l - 1; mm >= m; --mm) e *= sqrt((double)(l + mm + 1) / (double)(l - mm));
    if ((l - m) & 1) e = -e;
    double *Dl = D + wig_off(l);
    const int ld = l + 1;
    Dl[(int64_t)l * ld + m] = e;
    double prev = 0.0, cur = e;
    for (int k = l; k >= 1; --k) {
        const double nxt = (2.0 * m * cur - sqrt((double)(l - k) * (l + k + 1)) * prev) / sqrt((double)(l + k) * (l - k + 1));
        Dl[(int64_t)(k - 1) * ld + m] = nxt;
        prev = cur;
        cur = nxt;
    }
}

__device__ inline double Ieven(int q) { return 2.0 / (1.0 - (double)q * (double)q); }

// Folded table W^{m,p}[r, col] (row-major, ld = kc) for degree l = lstart(m,p) + 2r
// and m' = p + 2 col:  c_l sum_{k = l mod 2, k <= l} d^l_{k,0} d^l_{k,m} h(k, m', m),
// h = I(0) (k = 0, m' = 0), (1 + (-1)^m) I(k) (k > 0, m' = 0),
//     (1 + (-1)^m) I(m') (k = 0, m' > 0), 2 (I(k + m') + (-1)^m I(k - m')) otherwise.
__global__ void folded_table_kernel(int L, const double *__restrict__ D, double *W, int64_t blk, int kc)
{
    const int mp2 = blockIdx.y, m = mp2 >> 1, p = mp2 & 1;
    const int l0 = lstart(m, p);
    if (l0 >= L) return;
    const int R = (L - 1 - l0) / 2 + 1, Kc = p == 0 ? (L + 1) / 2 : L / 2;
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= (int64_t)R * Kc) return;
    const int r = (int)(g / Kc), col = (int)(g - (int64_t)r * Kc);
    const int l = l0 + 2 * r, mpr = p + 2 * col;
    const double sm = (m & 1) ? -1.0 : 1.0;
    const double *Dl = D + wig_off(l);
    const int ld = l + 1;
    double acc = 0.0;
    for (int k = l & 1; k <= l; k += 2) {
        double h;
        if (mpr == 0) h = (k == 0) ? Ieven(0) : (1.0 + sm) * Ieven(k);
        else h = (k == 0) ? (1.0 + sm) * Ieven(mpr) : 2.0 * (Ieven(k + mpr) + sm * Ieven(k - mpr));
        acc += Dl[(int64_t)k * ld] * Dl[(int64_t)k * ld + m] * h;
    }
    W[mp2 * blk + (int64_t)r * kc + col] = sqrt((2.0 * l + 1.0) / (4.0 * M_PI)) * acc;
}

// S table S^{m,p}[r', col] (row-major, ld = rc) for m' = p + 2r' and degree
// l = lstart(m,p) + 2 col: 2 pi c_l d^l_{m',0} d^l_{m',m} (zero for m' > l).
__global__ void s_table_kernel(int L, const double *__restrict__ D, double *S, int64_t blk, int rc)
{
    const int mp2 = blockIdx.y, m = mp2 >> 1, p = mp2 & 1;
    const int l0 = lstart(m, p);
    if (l0 >= L) return;
    const int R = (L - 1 - l0) / 2 + 1, Kr = p == 0 ? (L + 1) / 2 : L / 2;
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= (int64_t)R * Kr) return;
    const int rp = (int)(g / R), col = (int)(g - (int64_t)rp * R);
    const int l = l0 + 2 * col, mpr = p + 2 * rp;
    double v = 0.0;
    if (mpr <= l) {
        const double *Dl = D + wig_off(l);
        v = 2.0 * M_PI * sqrt((2.0 * l + 1.0) / (4.0 * M_PI)) * Dl[(int64_t)mpr * (l + 1)] * Dl[(int64_t)mpr * (l + 1) + m];
    }
    S[mp2 * blk + (int64_t)rp * rc + col] = v;
}

// Forward table A^{m,p}[j'][r] (column-major, ld = arows): the folded table
// composed with the colatitude DFT of the extended G_m,
//   a_{l,j'} = (1 / M) sum_{m' = p mod 2} W^{m,p}[r][m'/2] kap_{m mod 2}[m'][j'],
// kap_0 = 1 at the pole row, 2 cos(m' theta_j') elsewhere; kap_1 = 0 at the pole,
// 2 sin(m' theta_j') elsewhere (the -i of odd orders goes to the epilogue).  The
// equator column of rows with l + m odd is exactly zero.
__global__ void compose_forward_kernel(int L, int ntheta, const double *__restrict__ W, int64_t wblk, int kc,
                                       const double *__restrict__ kap, double *Af, const int64_t *__restrict__ aoff,
                                       const int *__restrict__ arows)
{
    const int mp2 = blockIdx.y, m = mp2 >> 1, p = mp2 & 1;
    const int l0 = lstart(m, p);
    if (l0 >= L) return;
    const int H = (ntheta + 1) / 2, M = 2 * ntheta - 2;
    const int R = (L - 1 - l0) / 2 + 1, Kc = p == 0 ? (L + 1) / 2 : L / 2;
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= (int64_t)R * H) return;
    const int jp = (int)(g / R), r = (int)(g - (int64_t)jp * R);
    double v = 0.0;
    if (!((ntheta & 1) && jp == H - 1 && ((p + m) & 1))) {
        const double *w = W + mp2 * wblk + (int64_t)r * kc;
        const double *kp = kap + ((int64_t)(m & 1) * L) * H + jp;
        for (int col = 0; col < Kc; ++col) v += w[col] * kp[(int64_t)(p + 2 * col) * H];
        v /= M;
    }
    Af[aoff[mp2] + (int64_t)jp * arows[mp2] + r] = v;
}

// Inverse table V^{m,p}[r][j'] (column-major over j', ld = ldv): the S table
// composed with the colatitude synthesis G_m(theta) = sum_m' K_{m,m'} e^{i m' theta},
//   v_{j',l} = sum_{m' = p mod 2} S^{m,p}[m'/2][r] lam_{m mod 2}[m'][j'],
// lam_0 = 1 (m' = 0), 2 cos(m' theta_j'); lam_1 = 0 (m' = 0), 2 sin(m' theta_j')
// (the i of odd orders goes to the longitude kernel).
__global__ void compose_inverse_kernel(int L, int ntheta, const double *__restrict__ S, int64_t sblk, int rc,
                                       const double *__restrict__ lam, double *V, const int64_t *__restrict__ voff,
                                       int64_t ldv)
{
    const int mp2 = blockIdx.y, m = mp2 >> 1, p = mp2 & 1;
    const int l0 = lstart(m, p);
    if (l0 >= L) return;
    const int H = (ntheta + 1) / 2;
    const int R = (L - 1 - l0) / 2 + 1, Kr = p == 0 ? (L + 1) / 2 : L / 2;
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= (int64_t)R * H) return;
    const int r = (int)(g / H), jp = (int)(g - (int64_t)r * H);
    const double *sp = S + mp2 * sblk + r;
    const double *lp = lam + ((int64_t)(m & 1) * L) * H + jp;
    double v = 0.0;
    for (int rp = 0; rp < Kr; ++rp) v += sp[(int64_t)rp * rc] * lp[(int64_t)(p + 2 * rp) * H];
    V[voff[mp2] + (int64_t)r * ldv + jp] = v;
}

}  // namespace sht
}  // namespace mpc

using namespace mpc;
using namespace mpc::sht;

// ---------------------------------------------------------------------- object
struct mpchol_sht {
    int dev = 0;
    hipStream_t st = nullptr;
    int L = 0, nth = 0, nph = 0, H = 0, tmax = 0, tmaxpad = 0;
    int kph = 0;      // forward K extent: H padded to GBK
    int64_t vrows = 0; // inverse row extent: H padded to GBM
    int nseq = 1;
    Plan Pphi{};
    double2 *tw = nullptr;
    double *Af = nullptr, *V = nullptr;               // composed tables
    int64_t *a_off = nullptr, *v_off = nullptr, *z_off = nullptr;
    int *a_rows = nullptr, *z_kpad = nullptr;
    Item *items_f = nullptr, *items_i = nullptr;
    int nitems_f = 0, nitems_i = 0;
    double *Gb = nullptr, *Bz = nullptr, *Ob = nullptr;  // work: folded G, packed z, GEMM results
    int *chunk_l = nullptr;                              // degree chunks of the f transposes
    int nchunk = 0, TT = 1, CH = 0;
    int64_t ldb = 0, gblk = 0, oblk = 0;
    size_t table_bytes = 0, work_bytes = 0;
};

namespace {

thread_local char g_sht_error[256] = "";

// Fewest passes with radices up to 12; of these the largest smallest radix (it
// sets the threads of a workgroup).
struct PlanSearch {
    Plan best{};
    int cur[MAXP];
    void go(int r, int from, int depth)
    {
        static const int radices[] = {12, 10, 9, 8, 6, 5, 4, 3, 2};
        if (r == 1) {  // nonincreasing: the last is the smallest
            if (best.np == 0 || depth < best.np || (depth == best.np && cur[depth - 1] > best.r[depth - 1])) {
                best.np = depth;
                std::copy(cur, cur + depth, best.r);
            }
            return;
        }
        if (depth == MAXP || (best.np && depth >= best.np)) return;
        for (int i = from; i < (int)(sizeof(radices) / sizeof(radices[0])); ++i)
            if (r % radices[i] == 0) {
                cur[depth] = radices[i];
                go(r / radices[i], i, depth + 1);
            }
    }
};
bool make_plan(int n, Plan &P)
{
    PlanSearch s;
    if (n == 1) {
        s.best.np = 1;
        s.best.r[0] = 1;
    } else {
        s.go(n, 0, 0);
    }
    P = s.best;
    P.n = n;
    return P.np > 0;
}

size_t fft_smem(int n, int nseq) { return ((size_t)nseq * seq_len(n) + n) * sizeof(double2); }
int fft_threads(const Plan &P, int nseq)
{
    int t = 1;
    for (int p = 0; p < P.np; ++p) {
        const int mb = butterflies(P.r[p]);
        t = std::max(t, (nseq * (P.n / P.r[p]) + mb - 1) / mb);
    }
    return (t + 63) / 64 * 64;  // at most 1024 for every length up to MAXN
}

// Sequences of a workgroup: a power of two (aligned runs of the blocks' rows) of
// at most eight, 512 threads and half of the LDS, so that two share a compute unit.
int fft_sequences(const Plan &P)
{
    int k = MAXSEQ;
    while (k > 1 && (fft_threads(P, k) > 512 || fft_smem(P.n, k) > 80 * 1024 - 512)) k /= 2;
    return k;
}

// e^{-2 pi i k / n}, exact at multiples of n/4, reduced to the first half turn.
std::vector<double2> twiddles(int n)
{
    std::vector<double2> w(n);
    for (int k = 0; k < n; ++k) {
        double c, s;
        if ((4 * (int64_t)k) % n == 0) {
            const int q = (int)((4 * (int64_t)k) / n);
            const double cs[4][2] = {{1, 0}, {0, -1}, {-1, 0}, {0, 1}};
            c = cs[q][0];
            s = cs[q][1];
        } else if (2 * k < n) {
            const double a = 2.0 * M_PI * (double)k / (double)n;
            c = std::cos(a);
            s = -std::sin(a);
        } else {
            const double a = 2.0 * M_PI * (double)(n - k) / (double)n;
            c = std::cos(a);
            s = std::sin(a);
        }
        w[k] = make_double2(c, s);
    }
    return w;
}

// cos(k pi x / y) and sin(k pi x / y) with the argument reduced exactly to
// [0, pi/2] through integer arithmetic (x k mod 2y).
void cossin_pi_ratio(int64_t num, int64_t den, double &c, double &s)
{
    int64_t a = num % (2 * den);  // angle = pi a / den in [0, 2 pi)
    double sc = 1.0, ss = 1.0;
    if (a >= den) {  // pi + b: cos -> -cos, sin -> -sin
        a -= den;
        sc = -sc;
        ss = -ss;
    }
    if (2 * a > den) {  // pi - b: cos -> -cos, sin -> sin
        a = den - a;
        sc = -sc;
    }
    if (a == 0) {
        c = sc;
        s = 0.0;
    } else if (2 * a == den) {
        c = 0.0;
        s = ss;
    } else {
        const double ang = M_PI * (double)a / (double)den;
        c = sc * std::cos(ang);
        s = ss * std::sin(ang);
    }
}

int rup(int x, int a) { return (x + a - 1) / a * a; }
int64_t rup64(int64_t x, int64_t a) { return (x + a - 1) / a * a; }

template <typename T> int dmalloc(T **p, size_t bytes, size_t &acc)
{
    if (hipMalloc((void **)p, bytes ? bytes : 16) != hipSuccess) {
        (void)hipGetLastError();
        *p = nullptr;
        return MPCHOL_ENOMEM;
    }
    acc += bytes;
    return MPCHOL_OK;
}

template <typename T> int upload(T *d, const std::vector<T> &h, hipStream_t st)
{
    if (h.empty()) return MPCHOL_OK;
    return hipMemcpyAsync(d, h.data(), h.size() * sizeof(T), hipMemcpyHostToDevice, st) == hipSuccess ? MPCHOL_OK
                                                                                                      : MPCHOL_EHIP;
}

// Raise a kernel's dynamic-LDS limit to at least `bytes` (never lower it: an
// object created earlier with larger transforms keeps launching).
void set_smem_attr(const void *k, size_t bytes)
{
    static std::vector<std::pair<const void *, size_t>> seen;
    static std::mutex mu;
    std::lock_guard<std::mutex> g(mu);
    for (auto &e : seen)
        if (e.first == k) {
            if (bytes <= e.second) return;
            e.second = bytes;
            (void)hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
            return;
        }
    seen.emplace_back(k, bytes);
    (void)hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

}  // namespace

extern "C" {

const char *mpchol_sht_last_error(void) { return g_sht_error; }

int mpchol_sht_destroy(mpchol_sht_t h)
{
    if (!h) return MPCHOL_OK;
    (void)hipSetDevice(h->dev);
    if (h->st) (void)hipStreamSynchronize(h->st);
    void *ps[] = {h->tw, h->Af, h->V, h->a_off, h->v_off, h->z_off, h->a_rows, h->z_kpad, h->items_f, h->items_i,
                  h->Gb, h->Bz, h->Ob, h->chunk_l};
    for (void *p : ps)
        if (p) (void)hipFree(p);
    delete h;
    return MPCHOL_OK;
}

int mpchol_sht_create(mpchol_sht_t *out, int32_t L, int32_t ntheta, int32_t nphi, int32_t tmax, int32_t device,
                      void *stream)
{
    if (!out) return MPCHOL_EINVAL;
    *out = nullptr;
    if (L < 1 || L > MAXL || ntheta < L + 1 || nphi < 2 * L - 1 || tmax < 1 || tmax > (1 << 20)) {
        snprintf(g_sht_error, sizeof(g_sht_error),
                 "invalid sizes: need 1 <= L <= %d, N_theta > L, N_phi >= 2L-1, 1 <= tmax <= 2^20", MAXL);
        return MPCHOL_EINVAL;
    }
    Plan Pphi;
    if (nphi > MAXN || !make_plan(nphi, Pphi)) {
        snprintf(g_sht_error, sizeof(g_sht_error), "FFT length N_phi = %d must be a product of 2, 3 and 5, at most %d",
                 nphi, MAXN);
        return MPCHOL_EINVAL;
    }
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || device < 0 || device >= ndev) {
        (void)hipGetLastError();
        snprintf(g_sht_error, sizeof(g_sht_error), "device %d not present", device);
        return MPCHOL_EHIP;
    }
    if (hipSetDevice(device) != hipSuccess) return MPCHOL_EHIP;
    mpchol_sht *h = new (std::nothrow) mpchol_sht();
    if (!h) return MPCHOL_ENOMEM;
    h->dev = device;
    h->st = (hipStream_t)stream;
    h->L = L;
    h->nth = ntheta;
    h->nph = nphi;
    h->H = (ntheta + 1) / 2;
    h->tmax = tmax;
    h->tmaxpad = rup(tmax, GBN / 2);
    h->Pphi = Pphi;
    h->nseq = fft_sequences(Pphi);
    h->ldb = 2 * (int64_t)h->tmaxpad;
    h->kph = rup(h->H, GBK);
    h->vrows = rup64(h->H, GBM);
    h->gblk = (int64_t)h->kph * h->ldb;
    h->oblk = h->vrows * h->ldb;
    const int H = h->H;

    // block geometry per (m, p): degrees l = lstart(m,p) + 2r, r < R
    const int nb = 2 * L;
    std::vector<int64_t> a_off(nb), v_off(nb), z_off(nb);
    std::vector<int> a_rows(nb), z_kpad(nb);
    std::vector<Item> items_f, items_i;
    const int kc = rup((L + 1) / 2, 2), rc = rup((L + 1) / 2, 2);  // row lengths of the temporary tables
    int64_t asz = 0, vsz = 0, zsz = 0;
    for (int m = 0; m < L; ++m)
        for (int p = 0; p < 2; ++p) {
            const int i = 2 * m + p, l0 = lstart(m, p);
            const int R = l0 < L ? (L - 1 - l0) / 2 + 1 : 0;
            a_rows[i] = rup(std::max(R, 1), GBM);
            a_off[i] = asz;
            asz += (int64_t)a_rows[i] * h->kph;
            z_kpad[i] = rup(std::max(R, 1), GBK);
            v_off[i] = vsz;
            vsz += (int64_t)z_kpad[i] * h->vrows;
            z_off[i] = zsz;
            zsz += (int64_t)z_kpad[i] * h->ldb;
        }
    // row blocks in the order in which the XCDs take them (runs of equal length):
    // every eighth (m, p) to one XCD, all of its row blocks together, so that the
    // K extents, which fall with m in the inverse, are the same for all XCDs
    for (int x = 0; x < 8; ++x)
        for (int i = x; i < nb; i += 8) {
            if (block_rows(L, i / 2, i % 2) == 0) continue;
            const int16_t m = (int16_t)(i / 2), p = (int16_t)(i % 2);
            for (int tm = 0; tm < a_rows[i] / GBM; ++tm) items_f.push_back(Item{m, p, tm});
            for (int tm = 0; tm < h->vrows / GBM; ++tm) items_i.push_back(Item{m, p, tm});
        }
    h->nitems_f = (int)items_f.size();
    h->nitems_i = (int)items_i.size();
    // f transposes: chunks of whole degrees of at most CH coefficients, TT time
    // steps per workgroup, TT * CH doubles of LDS (64 KB)
    h->CH = std::max(1024, rup(2 * L - 1, 256));
    h->TT = std::max(1, 8192 / h->CH);
    std::vector<int> chunk_l{0};
    for (int l = 0; l < L; ++l) {
        const int la = chunk_l.back();
        if ((l + 1) * (l + 1) - la * la > h->CH) chunk_l.push_back(l);
    }
    chunk_l.push_back(L);
    h->nchunk = (int)chunk_l.size() - 1;
    // colatitude weights of the composition, [m mod 2][m'][j']
    std::vector<double> kap(2 * (size_t)L * H), lam(2 * (size_t)L * H);
    for (int mp = 0; mp < L; ++mp)
        for (int jp = 0; jp < H; ++jp) {
            double c, s;
            cossin_pi_ratio((int64_t)mp * jp, ntheta - 1, c, s);  // m' theta_j' = pi m' j' / (N_theta - 1)
            const size_t e = (size_t)mp * H + jp, o = (size_t)L * H + e;
            kap[e] = jp == 0 ? 1.0 : 2.0 * c;
            kap[o] = jp == 0 ? 0.0 : 2.0 * s;
            lam[e] = mp == 0 ? 1.0 : 2.0 * c;
            lam[o] = mp == 0 ? 0.0 : 2.0 * s;
        }

    size_t tb = 0, wb = 0, scratch = 0;
    int rc_ = MPCHOL_OK;
    auto chk = [&](int r) {
        if (rc_ == MPCHOL_OK) rc_ = r;
    };
    double *D = nullptr, *Wt = nullptr, *St = nullptr, *kap_d = nullptr, *lam_d = nullptr;
    const int64_t wblk = (int64_t)rup((L + 1) / 2, 1) * kc, sblk = (int64_t)rup((L + 1) / 2, 1) * rc;
    chk(dmalloc(&h->tw, nphi * sizeof(double2), tb));
    chk(dmalloc(&h->Af, asz * 8, tb));
    chk(dmalloc(&h->V, vsz * 8, tb));
    chk(dmalloc(&h->a_off, nb * 8, tb));
    chk(dmalloc(&h->v_off, nb * 8, tb));
    chk(dmalloc(&h->z_off, nb * 8, tb));
    chk(dmalloc(&h->a_rows, nb * 4, tb));
    chk(dmalloc(&h->z_kpad, nb * 4, tb));
    chk(dmalloc(&h->items_f, std::max<size_t>(1, items_f.size()) * sizeof(Item), tb));
    chk(dmalloc(&h->items_i, std::max<size_t>(1, items_i.size()) * sizeof(Item), tb));
    chk(dmalloc(&h->Gb, (size_t)nb * h->gblk * 8, wb));
    chk(dmalloc(&h->Bz, zsz * 8, wb));
    chk(dmalloc(&h->Ob, (size_t)nb * h->oblk * 8, wb));
    chk(dmalloc(&h->chunk_l, chunk_l.size() * 4, tb));
    chk(dmalloc(&D, (size_t)wig_off(L) * 8, scratch));
    chk(dmalloc(&Wt, (size_t)nb * wblk * 8, scratch));
    chk(dmalloc(&St, (size_t)nb * sblk * 8, scratch));
    chk(dmalloc(&kap_d, kap.size() * 8, scratch));
    chk(dmalloc(&lam_d, lam.size() * 8, scratch));
    h->table_bytes = tb;
    h->work_bytes = wb;
    auto free_tmp = [&]() {
        void *ts[] = {D, Wt, St, kap_d, lam_d};
        for (void *p : ts)
            if (p) (void)hipFree(p);
    };
    if (rc_ != MPCHOL_OK) {
        snprintf(g_sht_error, sizeof(g_sht_error), "device allocation failed (tables %zu B, work %zu B)", tb, wb);
        free_tmp();
        mpchol_sht_destroy(h);
        return rc_;
    }
    hipStream_t st = h->st;
    // zero padding: padded K rows/columns of tables and operands must be zero,
    // and result blocks of (m, p) without any degree (m = L - 1, one parity)
    // are read as zero by the longitude kernel
    bool ok = hipMemsetAsync(h->Af, 0, asz * 8, st) == hipSuccess && hipMemsetAsync(h->V, 0, vsz * 8, st) == hipSuccess &&
              hipMemsetAsync(h->Gb, 0, (size_t)nb * h->gblk * 8, st) == hipSuccess &&
              hipMemsetAsync(h->Bz, 0, zsz * 8, st) == hipSuccess &&
              hipMemsetAsync(h->Ob, 0, (size_t)nb * h->oblk * 8, st) == hipSuccess;
    const std::vector<double2> twp = twiddles(nphi);
    if (ok)
        ok = upload(h->tw, twp, st) == MPCHOL_OK && upload(h->a_off, a_off, st) == MPCHOL_OK &&
             upload(h->v_off, v_off, st) == MPCHOL_OK && upload(h->z_off, z_off, st) == MPCHOL_OK &&
             upload(h->a_rows, a_rows, st) == MPCHOL_OK && upload(h->z_kpad, z_kpad, st) == MPCHOL_OK &&
             upload(h->items_f, items_f, st) == MPCHOL_OK && upload(h->items_i, items_i, st) == MPCHOL_OK &&
             upload(h->chunk_l, chunk_l, st) == MPCHOL_OK &&
             upload(kap_d, kap, st) == MPCHOL_OK && upload(lam_d, lam, st) == MPCHOL_OK;
    if (ok) {
        const int64_t nlm = (int64_t)L * (L + 1) / 2;
        wigner_kernel<<<(unsigned)((nlm + 255) / 256), 256, 0, st>>>(L, D);
        const int64_t half = (L + 1) / 2;
        dim3 gt((unsigned)((half * half + 255) / 256), (unsigned)nb);
        folded_table_kernel<<<gt, 256, 0, st>>>(L, D, Wt, wblk, kc);
        s_table_kernel<<<gt, 256, 0, st>>>(L, D, St, sblk, rc);
        dim3 gc((unsigned)((half * H + 255) / 256), (unsigned)nb);
        compose_forward_kernel<<<gc, 256, 0, st>>>(L, ntheta, Wt, wblk, kc, kap_d, h->Af, h->a_off, h->a_rows);
        compose_inverse_kernel<<<gc, 256, 0, st>>>(L, ntheta, St, sblk, rc, lam_d, h->V, h->v_off, h->vrows);
        ok = hipGetLastError() == hipSuccess && hipStreamSynchronize(st) == hipSuccess;
    }
    free_tmp();
    if (!ok) {
        snprintf(g_sht_error, sizeof(g_sht_error), "table set-up failed: %s", hipGetErrorString(hipGetLastError()));
        mpchol_sht_destroy(h);
        return MPCHOL_EHIP;
    }
    const size_t fs = fft_smem(nphi, h->nseq);
    set_smem_attr((const void *)phi_forward_kernel<512>, fs);
    set_smem_attr((const void *)phi_inverse_kernel<512>, fs);
    set_smem_attr((const void *)phi_forward_kernel<1024>, fs);
    set_smem_attr((const void *)phi_inverse_kernel<1024>, fs);
    set_smem_attr((const void *)gemm_forward_kernel<GBN, 2, 2>, SG<GBN, 2, 2>::SMEM);
    set_smem_attr((const void *)gemm_inverse_kernel<GBN, 2, 2>, SG<GBN, 2, 2>::SMEM);
    set_smem_attr((const void *)gemm_forward_kernel<16, 4, 1>, SG<16, 4, 1>::SMEM);
    set_smem_attr((const void *)gemm_inverse_kernel<16, 4, 1>, SG<16, 4, 1>::SMEM);
    set_smem_attr((const void *)unpack_forward_kernel, (size_t)h->TT * h->CH * 8);
    set_smem_attr((const void *)pack_inverse_kernel, (size_t)h->TT * h->CH * 8);
    *out = h;
    return MPCHOL_OK;
}

int mpchol_sht_info(mpchol_sht_t h, int64_t *table_bytes, int64_t *work_bytes, int64_t *gemm_flops_per_step)
{
    if (!h) return MPCHOL_EINVAL;
    if (table_bytes) *table_bytes = (int64_t)h->table_bytes;
    if (work_bytes) *work_bytes = (int64_t)h->work_bytes;
    if (gemm_flops_per_step) {
        // unpadded: per (m, p) degrees x northern colatitudes x 2 columns x 2 flops
        int64_t fl = 0;
        for (int m = 0; m < h->L; ++m)
            for (int p = 0; p < 2; ++p) {
                const int l0 = lstart(m, p);
                const int64_t R = l0 < h->L ? (h->L - 1 - l0) / 2 + 1 : 0;
                fl += 4 * R * h->H;
            }
        *gemm_flops_per_step = fl;
    }
    return MPCHOL_OK;
}

int mpchol_sht_forward(mpchol_sht_t h, const double *Z, int64_t T, double *f)
{
    if (!h || T < 0 || T > h->tmax) return MPCHOL_EINVAL;
    if (T == 0) return MPCHOL_OK;
    if (!Z || !f) return MPCHOL_EINVAL;
    if (hipSetDevice(h->dev) != hipSuccess) return MPCHOL_EHIP;
    hipStream_t st = h->st;
    const int64_t nsq = (int64_t)h->H * T;
    const unsigned gf = (unsigned)((nsq + h->nseq - 1) / h->nseq);
    const size_t fs = fft_smem(h->nph, h->nseq);
    auto phi = fft_threads(h->Pphi, h->nseq) <= 512 ? phi_forward_kernel<512> : phi_forward_kernel<1024>;
    phi<<<gf, fft_threads(h->Pphi, h->nseq), fs, st>>>(Z, (int)T, h->nth, h->L, h->Pphi, h->tw, h->Gb, h->gblk, h->ldb, h->nseq);
    auto gemm = [&](auto kernel, int bn, size_t smem) {
        const int ntn = (int)((2 * T + bn - 1) / bn);
        kernel<<<(unsigned)h->nitems_f * ntn, GNT, smem, st>>>(h->Af, h->a_off, h->a_rows, h->Gb, h->gblk, h->ldb,
                                                               h->kph, h->L, h->items_f, ntn, h->Ob, h->oblk);
    };
    if (T <= SMALL_T) gemm(gemm_forward_kernel<16, 4, 1>, 16, SG<16, 4, 1>::SMEM);
    else gemm(gemm_forward_kernel<GBN, 2, 2>, GBN, SG<GBN, 2, 2>::SMEM);
    dim3 gu((unsigned)h->nchunk, (unsigned)((T + h->TT - 1) / h->TT));
    unpack_forward_kernel<<<gu, TNT, (size_t)h->TT * h->CH * 8, st>>>(h->Ob, h->oblk, h->ldb, h->chunk_l, (int)T,
                                                                      h->L, h->TT, h->CH, f);
    return hipGetLastError() == hipSuccess ? MPCHOL_OK : MPCHOL_EHIP;
}

int mpchol_sht_inverse(mpchol_sht_t h, const double *f, int64_t T, double *Z)
{
    if (!h || T < 0 || T > h->tmax) return MPCHOL_EINVAL;
    if (T == 0) return MPCHOL_OK;
    if (!Z || !f) return MPCHOL_EINVAL;
    if (hipSetDevice(h->dev) != hipSuccess) return MPCHOL_EHIP;
    hipStream_t st = h->st;
    dim3 gp((unsigned)h->nchunk, (unsigned)((T + h->TT - 1) / h->TT));
    pack_inverse_kernel<<<gp, TNT, (size_t)h->TT * h->CH * 8, st>>>(f, h->chunk_l, (int)T, h->L, h->TT, h->CH, h->Bz,
                                                                    h->z_off, h->ldb);
    auto gemm = [&](auto kernel, int bn, size_t smem) {
        const int ntn = (int)((2 * T + bn - 1) / bn);
        kernel<<<(unsigned)h->nitems_i * ntn, GNT, smem, st>>>(h->V, h->v_off, h->vrows, h->z_kpad, h->Bz, h->z_off,
                                                               h->ldb, h->H, h->items_i, ntn, h->Ob, h->oblk);
    };
    if (T <= SMALL_T) gemm(gemm_inverse_kernel<16, 4, 1>, 16, SG<16, 4, 1>::SMEM);
    else gemm(gemm_inverse_kernel<GBN, 2, 2>, GBN, SG<GBN, 2, 2>::SMEM);
    const int64_t nsq = (int64_t)h->H * T;
    const unsigned gf = (unsigned)((nsq + h->nseq - 1) / h->nseq);
    auto phi = fft_threads(h->Pphi, h->nseq) <= 512 ? phi_inverse_kernel<512> : phi_inverse_kernel<1024>;
    phi<<<gf, fft_threads(h->Pphi, h->nseq), fft_smem(h->nph, h->nseq), st>>>(h->Ob, h->oblk, h->ldb, (int)T, h->nth, h->L,
                                                                    h->Pphi, h->tw, Z, h->nseq);
    return hipGetLastError() == hipSuccess ? MPCHOL_OK : MPCHOL_EHIP;
}

}  // extern "C"
