// Randomized estimate of the backward error ||Sigma - L L^T||_F: for probes
// V with independent N(0,1) entries, E ||E v||^2 = ||E||_F^2 (E symmetric), and
// E V = Sigma V - L (L^T V) costs O(N^2 k) instead of the N^3/3 of the exact
// residual.  Every stored tile is widened exactly to FP64 and read once per
// product; the products run on the FP64 MFMA.  Buffers have NT*b rows,
// identity beyond n.
//
// Sigma V for the generator with nondecreasing coordinates uses the
// exponential kernel's separability: with u_j = sigma_j v_j and
// d_i = exp(-(x_i - x_{i-1})/rho),
//   F_i = sum_{j<=i} e^{-(x_i-x_j)/rho} u_j = d_i F_{i-1} + u_i,
//   H_i = sum_{j>=i} e^{-(x_j-x_i)/rho} u_j = d_{i+1} H_{i+1} + u_i,
//   (Sigma v)_i = sigma_i (F_i + H_i - u_i) + nugget v_i,
// evaluated as a chunked scan (local recursions, chunk carries, combination).
// Otherwise (an explicit matrix, or unsorted coordinates) Sigma V is the
// dense product with Sigma regenerated or read from the kept copy.
#include "common.h"
#include "gemm_core.h"
#include "launch.h"

namespace mpc {

constexpr int EK = 64;   // probes per pass (columns of V)
constexpr int ER = 32;   // K rows staged per step
constexpr int SC = 256;  // rows per scan chunk

__device__ inline double source_ij(const Tiles &T, const Source &S, int64_t i, int64_t j)
{
    if (i >= T.n || j >= T.n) return (i == j) ? 1.0 : 0.0;
    if (S.orig) {
        int64_t a = i >= j ? i : j, c = i >= j ? j : i;  // lower part of the kept copy
        int I = (int)(a / T.b), J = (int)(c / T.b);
        return S.orig[tile_index(I, J) * (int64_t)T.b * T.b + (a % T.b) + (c % T.b) * (int64_t)T.b];
    }
    double v = S.sigma[i] * S.sigma[j] * exp(-fabs(S.x[i] - S.x[j]) / S.rho);
    if (i == j) v += S.nugget;
    return v;
}

// ---------------------------------------------------------------- dense Sigma V
// SV[i, q0+q] += sum_{j in chunk} Sigma_ij V[j, q0+q] for 32 probes; one
// thread per row i, 256 rows x 16384 columns per block, V staged 128 rows at
// a time.
constexpr int DQ = 32;
__global__ __launch_bounds__(256) void sigma_v_kernel(Tiles T, Source S, const double *V, int64_t ldv, double *SV)
{
    __shared__ double vs[128][DQ + 1];
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t j0 = (int64_t)blockIdx.y * 16384;
    const int64_t np = (int64_t)T.nt * T.b;
    double acc[DQ];
#pragma unroll
    for (int q = 0; q < DQ; ++q) acc[q] = 0.0;
    for (int64_t jc = j0; jc < j0 + 16384 && jc < np; jc += 128) {
        __syncthreads();
        for (int e = threadIdx.x; e < 128 * DQ; e += 256) {
            int jj = e % 128, q = e / 128;
            vs[jj][q] = (jc + jj < np) ? V[jc + jj + q * ldv] : 0.0;
        }
        __syncthreads();
        if (i < np) {
            for (int jj = 0; jj < 128 && jc + jj < np; ++jj) {
                double s = source_ij(T, S, i, jc + jj);
#pragma unroll
                for (int q = 0; q < DQ; ++q) acc[q] += s * vs[jj][q];
            }
        }
    }
    if (i < np)
#pragma unroll
        for (int q = 0; q < DQ; ++q) atomicAdd(SV + i + q * ldv, acc[q]);
}

// ---------------------------------------------------------------- scan Sigma V
// Local recursions of chunk c for probe q (rows s .. e, e < n):
//   f_i = d_i f_{i-1} + u_i (f_{s-1} = 0)   -> F buffer,
//   h_i = d_{i+1} h_{i+1} + u_i (h_{e+1} = 0) -> H buffer.
// F by the blocks of grid row 0, H by those of grid row 1.
__global__ __launch_bounds__(64) void scan_local_kernel(Tiles T, Source S, const double *__restrict__ V, int64_t ldv,
                                                        double *__restrict__ F, double *__restrict__ H)
{
    const int c = blockIdx.x, q = threadIdx.x;
    const int64_t s = (int64_t)c * SC, e = min((int64_t)T.n, s + SC) - 1;
    const double *v = V + q * ldv;
    if (blockIdx.y == 0) {
        double f = 0.0;
        for (int64_t i = s; i <= e; ++i) {
            const double d = (i > s) ? exp(-(S.x[i] - S.x[i - 1]) / S.rho) : 0.0;
            f = d * f + S.sigma[i] * v[i];
            F[i + q * ldv] = f;
        }
    } else {
        double h = 0.0;
        for (int64_t i = e; i >= s; --i) {
            const double d = (i < e) ? exp(-(S.x[i + 1] - S.x[i]) / S.rho) : 0.0;
            h = d * h + S.sigma[i] * v[i];
            H[i + q * ldv] = h;
        }
    }
}

// Chunk carries for probe q: Fin[c] = F_{s_c - 1} (block 0), Hin[c] = H_{e_c + 1}
// (block 1; both 0 at the ends), from the chunk-boundary values of the local
// recursions.
__global__ __launch_bounds__(64) void scan_carry_kernel(Tiles T, Source S, const double *__restrict__ F,
                                                        const double *__restrict__ H, int64_t ldv, int nchunk,
                                                        double *__restrict__ Fin, double *__restrict__ Hin)
{
    const int q = threadIdx.x;
    double carry = 0.0;
    if (blockIdx.x == 0) {  // F at the last row of the previous chunk
#pragma unroll 4
        for (int c = 0; c < nchunk; ++c) {
            const int64_t s = (int64_t)c * SC, e = min((int64_t)T.n, s + SC) - 1;
            Fin[c * EK + q] = carry;
            const double dc = (c > 0) ? exp(-(S.x[e] - S.x[s - 1]) / S.rho) : 0.0;
            carry = F[e + q * ldv] + dc * carry;
        }
    } else {  // H at the first row of the next chunk
#pragma unroll 4
        for (int c = nchunk - 1; c >= 0; --c) {
            const int64_t s = (int64_t)c * SC, e = min((int64_t)T.n, s + SC) - 1;
            Hin[c * EK + q] = carry;
            const double dc = (c < nchunk - 1) ? exp(-(S.x[e + 1] - S.x[s]) / S.rho) : 0.0;
            carry = H[s + q * ldv] + dc * carry;
        }
    }
}

// SV_i = sigma_i (F_i + H_i - u_i) + nugget v_i with the carries applied;
// rows >= n are the identity's.  F may alias SV (each element read, then written).
__global__ __launch_bounds__(256) void scan_finish_kernel(Tiles T, Source S, const double *V, int64_t ldv,
                                                          const double *F, const double *H, const double *Fin,
                                                          const double *Hin, double *SV)
{
    const int64_t np = (int64_t)T.nt * T.b;
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= np * EK) return;
    const int64_t i = e % np;
    const int q = (int)(e / np);
    const double v = V[i + q * ldv];
    if (i >= T.n) {
        SV[i + q * ldv] = v;
        return;
    }
    const int c = (int)(i / SC);
    const int64_t s = (int64_t)c * SC, ce = min((int64_t)T.n, s + SC) - 1;
    double Fi = F[i + q * ldv], Hi = H[i + q * ldv];
    if (c > 0) Fi += exp(-(S.x[i] - S.x[s - 1]) / S.rho) * Fin[c * EK + q];
    if (ce + 1 < T.n) Hi += exp(-(S.x[ce + 1] - S.x[i]) / S.rho) * Hin[c * EK + q];
    const double u = S.sigma[i] * v;
    SV[i + q * ldv] = S.sigma[i] * (Fi + Hi - u) + S.nugget * v;
}

// ---------------------------------------------------------------- L^T V, L W
// LT:  W[c of tile column K] = sum_{I >= K} L_IK(:, c)^T V[rows of I],
// !LT: Z[r of tile row I]    = sum_{K <= I} L_IK(r, :) W[rows of K]:
// strips of BM outputs (32 or 64), four waves of BM outputs x 16 probes, the sum taken ER
// rows (columns) of the stored tiles at a time on the FP64 MFMA.  What bounds it:
// the latency of the pieces, then the MFMA.  Two steps' pieces of L and probes are
// on their way in registers while a third is multiplied from LDS; they are widened
// only when staged, and no branch on the class stands between the loads.  A block
// takes a long strip and then the short one from the other end, so that all blocks
// are equally long.  All strips walk the probes from the same end, so that the L2
// serves each piece to the blocks that meet there.  (N = 32,768: 4.4 (LT) and
// 5.4 -> 2.1 ms each, 33 TFLOP/s.)
constexpr int QPT = ER * EK / 256;      // elements of the probe piece per thread
constexpr int LDK = ER + 2;  // 32 lanes of a read meet each of the 64 banks once
static_assert(ER * EK % 256 == 0, "staging split");

template <bool LT, int BM>
__global__ __launch_bounds__(256) void factor_apply_kernel(Tiles T, const double *__restrict__ X, int64_t ldx,
                                                           double *__restrict__ Y, int strips, bool pair)
{
    // LT: rows of a tile are the summed index, consecutive in memory and in LDS
    // (ls[c][r]); otherwise the outputs are (ls[k][r])
    constexpr int LDR = BM + 16;
    __shared__ __align__(16) double ls[2][LT ? BM * LDK : ER * LDR], xs[2][EK * LDK];
    constexpr int LPT = ER * BM / 256 / 2;  // row pairs of the L piece per thread
    static_assert(ER * BM % 512 == 0, "staging split");
    constexpr int MB = BM / 16, FAST = LT ? ER : BM;  // row index runs over FAST
    constexpr int COL = 2 * 256 / FAST;               // columns per round of loads
    const int b = T.b, per = b / BM, nrs = b / ER;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, gi = lane & 15, gg = lane >> 4;
    const int r2 = 2 * (tid % (FAST / 2)), c0 = tid / (FAST / 2);
    double4_t acc[MB];
#pragma unroll
    for (int m = 0; m < MB; ++m) acc[m] = (double4_t){0.0, 0.0, 0.0, 0.0};
    // strips in order of length; "far" tile rows (columns) from the longest
    const int sa = blockIdx.x, sb = strips - 1 - sa;
    const int na = (T.nt - sa / per) * nrs, nsteps = na + (pair ? (T.nt - sb / per) * nrs : 0);
    struct Step {  // one step's piece, on its way
        ulonglong2 l[LPT];
        double x[QPT];
        int cls, ts;
    } f0, f1;
    int next = 0;
    const double *xp = X + tid % ER + (int64_t)(tid / ER) * ldx;
    auto place = [&](int st, int &I, int &K, int &o0, int &k0) {  // step st: piece of tile (I, K)
        const bool first = st < na;
        const int strip = first ? sa : sb, s = first ? st : st - na;
        const int far = strip / per, w = s / nrs;
        o0 = (strip - far * per) * BM;
        k0 = (s - w * nrs) * ER;
        I = LT ? T.nt - 1 - w : T.nt - 1 - far;
        K = LT ? far : w;
    };
    auto class_at = [&](int st) {
        int I, K, o0, k0;
        place(min(st, nsteps - 1), I, K, o0, k0);
        return (I == K) ? (int)P64 : (int)T.map[I + (int64_t)K * T.nt];
    };
    auto fetch = [&](Step &f, int st) {
        int I, K, o0, k0;
        place(min(st, nsteps - 1), I, K, o0, k0);
        f.cls = __builtin_amdgcn_readfirstlane(next);  // read a step ahead
        next = class_at(st + 1);
        f.ts = T.tscale[I + (int64_t)K * T.nt];
        const char *tile = T.slots + tile_index(I, K) * T.slot_bytes;
        const int off = (LT ? k0 + r2 + (o0 + c0) * b : o0 + r2 + (k0 + c0) * b), sh = class_shift(f.cls);
#pragma unroll
        for (int j = 0; j < LPT; ++j) f.l[j] = load_pair16(tile, (off + COL * j * b) << sh);
        const double *x = xp + (int64_t)(LT ? I : K) * b + k0;
#pragma unroll
        for (int j = 0; j < QPT; ++j) f.x[j] = x[(int64_t)(256 / ER * j) * ldx];
    };
    auto put = [&](const Step &f, int buf) {
        // columns and strips start at multiples of 32 values: only the row pair places a value in its 16 bytes
        const int byte = r2 << class_shift(f.cls);
#pragma unroll
        for (int j = 0; j < LPT; ++j) {
            double d0, d1;
            if (f.cls == P64) {
                d0 = __longlong_as_double((long long)f.l[j].x);
                d1 = __longlong_as_double((long long)f.l[j].y);
            } else {
                const uint64_t u = pair_codes(f.l[j], byte);
                const uint32_t w = (uint32_t)u;
                if (f.cls == P32) {
                    d0 = (double)__uint_as_float(w);
                    d1 = (double)__uint_as_float((uint32_t)(u >> 32));
                } else if (f.cls == P16) {
                    d0 = decode_class(w & 0xFFFFu, P16, T.lo16, f.ts);
                    d1 = decode_class((w >> 16) & 0xFFFFu, P16, T.lo16, f.ts);
                } else {
                    d0 = decode_class(w & 0xFFu, P8, T.lo16, f.ts);
                    d1 = decode_class((w >> 8) & 0xFFu, P8, T.lo16, f.ts);
                }
            }
            *(double2 *)&ls[buf][(c0 + COL * j) * (LT ? LDK : LDR) + r2] = make_double2(d0, d1);
        }
#pragma unroll
        for (int j = 0; j < QPT; ++j) xs[buf][(tid / ER + 256 / ER * j) * LDK + tid % ER] = f.x[j];
    };
    auto store = [&](int strip) {
        const int far = strip / per, fixed = LT ? far : T.nt - 1 - far;
        double *y = Y + (int64_t)fixed * b + (strip - far * per) * BM + gi + (int64_t)(wave * 16) * ldx;
#pragma unroll
        for (int m = 0; m < MB; ++m)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                y[m * 16 + (int64_t)acc_row<double>(gg, v) * ldx] = acc[m][v];
                acc[m][v] = 0.0;
            }
    };
    auto multiply = [&](int buf) {
        const double *lc = ls[buf], *xc = xs[buf];
#pragma unroll
        for (int s = 0; s < ER / 4; ++s) {
            // swapped operands: lane gi owns output gi, element v the probe acc_row(gg, v)
            const double fx = xc[(wave * 16 + gi) * LDK + s * 4 + gg];
#pragma unroll
            for (int m = 0; m < MB; ++m) {
                const double fl = LT ? lc[(m * 16 + gi) * LDK + s * 4 + gg] : lc[(s * 4 + gg) * LDR + m * 16 + gi];
                acc[m] = __builtin_amdgcn_mfma_f64_16x16x4f64(fx, fl, acc[m], 0, 0, 0);
            }
        }
    };
    next = class_at(0);
    fetch(f0, 0);
    fetch(f1, 1);
    put(f0, 0);
    __syncthreads();
    for (int st = 0; st < nsteps; st += 2) {  // na and nsteps are even: b / ER is
        fetch(f0, st + 2);
        multiply(0);
        put(f1, 1);
        __syncthreads();
        fetch(f1, st + 3);
        multiply(1);
        if (st + 2 == na) store(sa);
        put(f0, 0);
        __syncthreads();
    }
    if (pair) store(sb);
}

// Pairs of strips where they still make two blocks per compute unit; with fewer
// strips the longest one decides, and single strips start them all at once.
template <bool LT, int BM>
static void factor_apply(const Tiles &T, const double *X, int64_t ldx, double *Y, hipStream_t st)
{
    const int strips = T.nt * (T.b / BM);  // even: b is a multiple of 128
    const bool pair = strips >= 1024;
    factor_apply_kernel<LT, BM><<<(unsigned)(pair ? strips / 2 : strips), 256, 0, st>>>(T, X, ldx, Y, strips, pair);
}

// Widen FP32 normals to FP64 probes, zero beyond n.
__global__ void probes_kernel(const float *z, int64_t n, int64_t np, double *V)
{
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= np * EK) return;
    const int64_t i = e % np, q = e / np;
    V[e] = (i < n) ? (double)z[i + q * n] : 0.0;
}

// sum over rows < n and probes of (SV - Z)^2 in a fixed order: the SC rows of a
// chunk by one block each, then the chunks' sums by one block (one block for
// all of it took 1.19 ms at N = 32,768).
__device__ inline double block_sum256(double a)
{
    __shared__ double s[256];
    s[threadIdx.x] = a;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) s[threadIdx.x] += s[threadIdx.x + w];
        __syncthreads();
    }
    return s[0];
}

__global__ __launch_bounds__(SC) void residual_part_kernel(const double *SV, const double *Z, int64_t n, int64_t np,
                                                           double *part)
{
    const int64_t i = (int64_t)blockIdx.x * SC + threadIdx.x;
    double a = 0.0;
    if (i < n)
#pragma unroll 8
        for (int q = 0; q < EK; ++q) {
            const double d = SV[i + q * np] - Z[i + q * np];
            a += d * d;
        }
    a = block_sum256(a);
    if (threadIdx.x == 0) part[blockIdx.x] = a;
}

__global__ __launch_bounds__(256) void residual_sum_kernel(const double *part, int nparts, double *out)
{
    double a = 0.0;
    for (int p = threadIdx.x; p < nparts; p += 256) a += part[p];
    a = block_sum256(a);
    if (threadIdx.x == 0) *out = a;
}

int estimate_chunks(int64_t n) { return (int)((n + SC - 1) / SC); }

// scratch: 3 * NT*b*EK doubles + 2 * chunks*EK doubles; zbuf: n*EK floats.
// Writes sum ||E v_q||^2 over the EK probes to *out (device).  sorted: the
// generator's coordinates are nondecreasing (scan path for Sigma V).
void launch_estimate(const Tiles &T, const Source &S, bool sorted, uint64_t seed, double *scratch, float *zbuf,
                     double *out, hipStream_t st)
{
    const int64_t np = (int64_t)T.nt * T.b;
    double *V = scratch, *SV = scratch + np * EK, *W = scratch + 2 * np * EK, *Z = scratch;  // Z reuses V
    double *Fin = scratch + 3 * np * EK, *Hin = Fin + (int64_t)estimate_chunks(T.n) * EK;
    launch_normal_matrix(seed, T.n, EK, zbuf, T.n, st);
    const unsigned eb = (unsigned)((np * EK + 255) / 256);
    probes_kernel<<<eb, 256, 0, st>>>(zbuf, T.n, np, V);
    if (sorted && !S.orig) {
        const int nc = estimate_chunks(T.n);
        scan_local_kernel<<<dim3(nc, 2), EK, 0, st>>>(T, S, V, np, SV, W);  // F -> SV, H -> W
        scan_carry_kernel<<<2, EK, 0, st>>>(T, S, SV, W, np, nc, Fin, Hin);
        scan_finish_kernel<<<eb, 256, 0, st>>>(T, S, V, np, SV, W, Fin, Hin, SV);
    } else {
        (void)hipMemsetAsync(SV, 0, (size_t)np * EK * 8, st);
        const dim3 g((unsigned)((np + 255) / 256), (unsigned)((np + 16383) / 16384));
        for (int q0 = 0; q0 < EK; q0 += DQ) sigma_v_kernel<<<g, 256, 0, st>>>(T, S, V + q0 * np, np, SV + q0 * np);
    }
    // strips of 64 halve the readings of the probes, but few of them leave the GPU
    // uneven (both products, strips of 32 and 64: N = 32,768 4.2 and 5.6 ms, 49,152
    // 9.2 and 8.9, 65,536 16.0 and 13.8, 129,600 60.5 and 54.8)
    if (np >= 49152) {
        factor_apply<true, 64>(T, V, np, W, st);
        factor_apply<false, 64>(T, W, np, Z, st);
    } else {
        factor_apply<true, 32>(T, V, np, W, st);
        factor_apply<false, 32>(T, W, np, Z, st);
    }
    residual_part_kernel<<<estimate_chunks(T.n), SC, 0, st>>>(SV, Z, T.n, np, Fin);
    residual_sum_kernel<<<1, 256, 0, st>>>(Fin, estimate_chunks(T.n), out);
}

int estimate_probes() { return EK; }

}  // namespace mpc
