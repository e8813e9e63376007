// Tile-level elementwise kernels: covariance generation and loading, tile
// norms, the sender-side conversion of a factored panel, log-determinant
// reduction and factor export.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "launch.h"

namespace mpc {

// Sigma at row r, column c of tile (I, J); identity in the padding beyond n.
__device__ inline double source_value(const Tiles &T, const Source &S, int I, int J, int r, int c)
{
    int64_t i = (int64_t)I * T.b + r, j = (int64_t)J * T.b + c;
    if (i >= T.n || j >= T.n) return (i == j) ? 1.0 : 0.0;
    if (S.dense) return i >= j ? S.dense[i + j * S.ld] : S.dense[j + i * S.ld];
    if (S.orig) return S.orig[tile_index(I, J) * (int64_t)T.b * T.b + r + (int64_t)c * T.b];
    double v = S.sigma[i] * S.sigma[j] * exp(-fabs(S.x[i] - S.x[j]) / S.rho);
    if (i == j) v += S.nugget;
    return v;
}

// Elementwise walks of a tile: 128 consecutive rows per column and two (norms:
// eight) columns at a time, so that no element index is divided by the tile size.

// Frobenius norm squared and max |.| of the valid part of every lower tile:
// `parts` blocks per tile, each a run of its columns, fixed-order reduction
// (deterministic).  One part: straight into fro2 and amax; else into
// partial[t * 2 * parts + part] and, parts further on, the maximum.  Bound by the
// exponentials of the generator, or by the bytes of a matrix; a single block per
// tile left most compute units idle (N = 16,384: 0.57 -> 0.39 ms, N = 1,024: 57 ->
// 16 us, a matrix of N = 8,100: 0.51 -> 0.10 ms).
__global__ __launch_bounds__(1024) void norms_kernel(Tiles T, Source S, int parts, double *partial, double *fro2,
                                                     double *amax)
{
    __shared__ double ss[1024], sm[1024];
    int I, J;
    const int t = blockIdx.x / parts, part = blockIdx.x % parts;
    tile_ij(t, I, J);
    const int b = T.b, tid = threadIdx.x;
    double s = 0.0, m = 0.0;
    const int rmax = (int)min((int64_t)b, T.n - (int64_t)I * b), cmax = (int)min((int64_t)b, T.n - (int64_t)J * b);
    const int cb = part * b / parts, c1 = min(cmax, (part + 1) * b / parts);
    for (int r = tid % 128; r < rmax; r += 128)
#pragma unroll 2
        for (int c = cb + tid / 128; c < c1; c += 8) {
            double v = source_value(T, S, I, J, r, c);
            s += v * v;
            m = fmax(m, fabs(v));
        }
    ss[tid] = s;
    sm[tid] = m;
    __syncthreads();
    for (int w = 512; w > 0; w >>= 1) {
        if (tid < w) {
            ss[tid] += ss[tid + w];
            sm[tid] = fmax(sm[tid], sm[tid + w]);
        }
        __syncthreads();
    }
    if (tid == 0) {
        const bool direct = parts == 1;
        *(direct ? fro2 + I + (int64_t)J * T.nt : partial + (int64_t)t * 2 * parts + part) = ss[0];
        *(direct ? amax + I + (int64_t)J * T.nt : partial + (int64_t)t * 2 * parts + parts + part) = sm[0];
    }
}

__global__ __launch_bounds__(256) void norms_reduce_kernel(int nt, int64_t ntile, int parts, const double *partial,
                                                           double *fro2, double *amax)
{
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t >= ntile) return;
    int I, J;
    tile_ij(t, I, J);
    double s = 0.0, m = 0.0;
    for (int p = 0; p < parts; ++p) {
        s += partial[t * 2 * parts + p];
        m = fmax(m, partial[t * 2 * parts + parts + p]);
    }
    fro2[I + (int64_t)J * nt] = s;
    amax[I + (int64_t)J * nt] = m;
}

// Write Sigma into the work tiles: FP64 for FP64-class and diagonal tiles,
// FP32 (rounded to nearest) for every lower class.  Blocks of 128 rows by 16 columns.
__global__ __launch_bounds__(256) void load_kernel(Tiles T, Source S)
{
    int I, J;
    tile_ij(blockIdx.y, I, J);
    const int b = T.b, nr = b / 128;
    const int cls = (I == J) ? P64 : T.map[I + (int64_t)J * T.nt];
    char *slot = T.slots + tile_index(I, J) * T.slot_bytes;
    const int r = (int)(blockIdx.x % nr) * 128 + (int)threadIdx.x % 128;
    const int c0 = (int)(blockIdx.x / nr) * 16 + (int)threadIdx.x / 128;
#pragma unroll
    for (int c = c0; c < c0 + 16; c += 2) {
        const double v = source_value(T, S, I, J, r, c);
        if (cls == P64) ((double *)slot)[r + c * b] = v;
        else ((float *)slot)[r + c * b] = (float)v;
    }
}

// Copy a caller matrix (column-major, lower part read) into FP64 tiles in the
// packed layout; diagonal tiles are filled symmetrically from their lower part.
__global__ __launch_bounds__(256) void copy_matrix_kernel(Tiles T, const double *A, int64_t lda, double *orig)
{
    int I, J;
    tile_ij(blockIdx.y, I, J);
    const int b = T.b, nr = b / 128;
    double *dst = orig + tile_index(I, J) * (int64_t)b * b;
    const int r = (int)(blockIdx.x % nr) * 128 + (int)threadIdx.x % 128;
    const int c0 = (int)(blockIdx.x / nr) * 16 + (int)threadIdx.x / 128;
    const int64_t i = (int64_t)I * b + r;
#pragma unroll
    for (int c = c0; c < c0 + 16; c += 2) {
        const int64_t j = (int64_t)J * b + c;
        double v = 0.0;
        if (i < T.n && j < T.n) v = (i >= j) ? A[i + j * lda] : A[j + i * lda];
        dst[r + c * b] = v;
    }
}

// Sender-side conversion of step k (one 64 x 64 sub-tile per block).
// The TRSM output X (FP64, in p64[I]) becomes the stored value S of tile
// (I,k) in its class -- FP64: X; FP32: (float)X; 16-bit/FP8: the scaled,
// rounded code of (float)X with t from max|(float)X| -- and every class q
// in qmask[I] gets its copy: FP64 S, FP32 (float)S (or, with the split
// products, its three BF16 parts), 16-bit/FP8 the code of S with the copy's
// own scale (row-major for the 16-bit, 8-bit and split copies).  With
// block-scaled FP8 (lo8 MX) every 32 columns of a row of the FP8 copy take
// their own scale from their own largest |S|, written as the E8M0 byte 127 - t.
__global__ __launch_bounds__(256) void convert_kernel(Tiles T, Panel P, int k, const uint8_t *qmask)
{
    __builtin_amdgcn_s_setprio(3);  // the panel chain: issue ahead of update waves sharing the SIMD
    __shared__ double xs[64][65];  // xs[c][r]
    __shared__ int xt[64][2];      // lo8 MX: scale exponent of row r, 32-column half h of the sub-tile
    const int b = T.b, nsub = b / 64;
    const int I = k + 1 + blockIdx.y;
    const int sr = blockIdx.x % nsub, sc = blockIdx.x / nsub;
    const int64_t bb = (int64_t)b * b;
    const int cls = T.map[I + (int64_t)k * T.nt];
    const int lo16 = T.lo16;
    const uint8_t mask = qmask[I];
    if (panel_direct(cls, mask)) return;
    double *x64 = P.p64 + (int64_t)I * bb;
    char *slot = T.slots + tile_index(I, k) * T.slot_bytes;

    const double m = __longlong_as_double((long long)P.pmax[I]);
    int ts = 0;
    double mS = m;
    if (cls == P32) mS = (double)(float)m;
    else if (cls >= P16) {
        double mf = (double)(float)m;
        ts = scale_exp(mf, cls, lo16);
        mS = decode_class(encode_class(mf, cls, lo16, ts), cls, lo16, ts);
    }
    int tq[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) tq[q] = scale_exp(mS, q, lo16);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        T.tscale[I + (int64_t)k * T.nt] = ts;
        for (int q = 0; q < 4; ++q) P.pscale[I * 4 + q] = tq[q];
    }

    // 16 values a thread, all read before the first is used
    const int r = threadIdx.x & 63, c0 = threadIdx.x >> 6;
    const int off0 = sr * 64 + r + (sc * 64 + c0) * b;  // within one tile
    double X[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) X[j] = x64[off0 + 4 * j * b];
    auto store = [&](auto q) {
        constexpr int CLS = decltype(q)::value;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int off = off0 + 4 * j * b;
            double Sv = X[j];
            if (CLS == P64) {
                ((double *)slot)[off] = Sv;
            } else if (CLS == P32) {
                const float f = (float)X[j];
                Sv = (double)f;
                ((float *)slot)[off] = f;
            } else {
                const uint32_t code = encode_class((double)(float)X[j], CLS, lo16, ts);
                Sv = decode_class(code, CLS, lo16, ts);
                if (CLS == P16) ((uint16_t *)slot)[off] = (uint16_t)code;
                else ((uint8_t *)slot)[off] = (uint8_t)code;
            }
            xs[c0 + 4 * j][r] = Sv;
            if (mask & 1) x64[off] = Sv;
            if ((mask & 2) && !T.lo32) P.p32[(int64_t)I * bb + off] = (float)Sv;
        }
    };
    switch (cls) {
    case P64: store(std::integral_constant<int, P64>{}); break;
    case P32: store(std::integral_constant<int, P32>{}); break;
    case P16: store(std::integral_constant<int, P16>{}); break;
    default: store(std::integral_constant<int, P8>{}); break;
    }
    const bool split = (mask & 2) && T.lo32;
    const bool mx = (mask & 8) && T.lo8;
    if ((mask & 12) || split) {
        __syncthreads();
        if (mx) {
            if (threadIdx.x < 128) {
                const int r = threadIdx.x & 63, h = threadIdx.x >> 6;
                double a = 0.0;
                for (int c = 0; c < 32; ++c) a = fmax(a, fabs(xs[h * 32 + c][r]));
                const int t = min(max(scale_exp(a, P8, lo16), -127), 127);  // 0 for an all-zero block
                xt[r][h] = t;
                P.p8x[(int64_t)I * (bb / 32) + (int64_t)(sr * 64 + r) * (b / 32) + sc * 2 + h] = (uint8_t)(127 - t);
            }
            __syncthreads();
        }
        // four consecutive columns of a row per thread and round: whole words out
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int c = 4 * (threadIdx.x & 15), rr = (threadIdx.x >> 4) + 16 * j;
            const int64_t roff = (int64_t)I * bb + (int64_t)(sr * 64 + rr) * b + (sc * 64 + c);
            double Sv[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) Sv[i] = xs[c + i][rr];
            if (mask & 4) {
                uint32_t u[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) u[i] = encode_class(Sv[i], P16, lo16, tq[P16]);
                *(uint2 *)(P.p16 + roff) = make_uint2(u[0] | u[1] << 16, u[2] | u[3] << 16);
            }
            if (mask & 8) {
                const int t = mx ? xt[rr][c >> 5] : tq[P8];
                uint32_t u[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) u[i] = encode_class(Sv[i], P8, lo16, t);
                *(uint32_t *)(P.p8 + roff) = u[0] | u[1] << 8 | u[2] << 16 | u[3] << 24;
            }
            if (split) {  // FP32 copy as hi + mid + lo, each step exact in FP32
                uint32_t hi[4], mid[4], lo[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float f = (float)Sv[i];
                    hi[i] = f32_to_bf16(f);
                    const float r1 = f - bf16_to_f32((uint16_t)hi[i]);
                    mid[i] = f32_to_bf16(r1);
                    lo[i] = f32_to_bf16(r1 - bf16_to_f32((uint16_t)mid[i]));
                }
                uint16_t *d = P.p32s + (int64_t)I * 2 * bb + roff;  // roff holds I * bb already
                *(uint2 *)d = make_uint2(hi[0] | hi[1] << 16, hi[2] | hi[3] << 16);
                *(uint2 *)(d + bb) = make_uint2(mid[0] | mid[1] << 16, mid[2] | mid[3] << 16);
                *(uint2 *)(d + 2 * bb) = make_uint2(lo[0] | lo[1] << 16, lo[2] | lo[3] << 16);
            }
        }
    }
}

// 2 * sum_i log L_ii over i < n, one block, fixed-order reduction.
__global__ __launch_bounds__(1024) void logdet_kernel(Tiles T, double *out)
{
    __shared__ double s[1024];
    double acc = 0.0;
    for (int64_t i = threadIdx.x; i < T.n; i += 1024) {
        int K = (int)(i / T.b), r = (int)(i % T.b);
        const double *d = (const double *)(T.slots + tile_index(K, K) * T.slot_bytes);
        acc += log(d[r + (int64_t)r * T.b]);
    }
    s[threadIdx.x] = acc;
    __syncthreads();
    for (int w = 512; w > 0; w >>= 1) {
        if (threadIdx.x < w) s[threadIdx.x] += s[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = 2.0 * s[0];
}

// Dense copy of the factor's represented values (strict upper part zero): 128
// rows by 16 columns per block, all in one tile, two rows a thread and column.
// What bounds it: memory (a value at a time behind a branch on the class, N = 16,384:
// 935 -> 546 us, 5.9 TB/s).  WIDE: L and its columns lie on 16 bytes.
template <int CLS, bool WIDE>
__device__ inline void copy_block(const char *slot, int b, int lo16, int ts, int lr, int lc, int64_t i, int64_t j0,
                                  int64_t n, double *L, int64_t ldl)
{
    ulonglong2 raw[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) raw[q] = load_pair16(slot, (lr + (lc + 4 * q) * b) << class_shift(CLS));
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int64_t j = j0 + 4 * q;
        double v0, v1;
        if (CLS == P64) {
            v0 = __longlong_as_double((long long)raw[q].x);
            v1 = __longlong_as_double((long long)raw[q].y);
        } else {
            constexpr int BITS = CLS == P32 ? 32 : CLS == P16 ? 16 : 8;
            constexpr uint32_t MASK = BITS == 32 ? ~0u : (1u << (BITS & 31)) - 1;
            const uint64_t u = pair_codes(raw[q], lr << class_shift(CLS));
            v0 = decode_class((uint32_t)u & MASK, CLS, lo16, ts);
            v1 = decode_class((uint32_t)(u >> BITS) & MASK, CLS, lo16, ts);
        }
        if (i < j) v0 = 0.0;
        if (i + 1 < j) v1 = 0.0;
        if (j >= n) continue;
        double *d = L + i + j * ldl;
        if (WIDE && i + 1 < n) {
            *(double2 *)d = make_double2(v0, v1);
        } else {
            if (i < n) d[0] = v0;
            if (i + 1 < n) d[1] = v1;
        }
    }
}

template <bool WIDE>
__global__ __launch_bounds__(256) void get_factor_kernel(Tiles T, double *L, int64_t ldl)
{
    const int b = T.b;
    const int64_t i0 = (int64_t)blockIdx.x * 128, c0 = (int64_t)blockIdx.y * 16;
    const int64_t i = i0 + 2 * (threadIdx.x & 63), j0 = c0 + (threadIdx.x >> 6);
    if (i0 + 127 < c0) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int64_t j = j0 + 4 * q;
            if (j >= T.n) break;
            double *d = L + i + j * ldl;
            if (WIDE && i + 1 < T.n) {
                *(double2 *)d = make_double2(0.0, 0.0);
            } else {
                if (i < T.n) d[0] = 0.0;
                if (i + 1 < T.n) d[1] = 0.0;
            }
        }
        return;
    }
    const int I = (int)(i0 / b), J = (int)(c0 / b), lr = (int)(i - (int64_t)I * b), lc = (int)(j0 - (int64_t)J * b);
    const int cls = I == J ? (int)P64 : (int)T.map[I + (int64_t)J * T.nt], ts = T.tscale[I + (int64_t)J * T.nt];
    const char *slot = T.slots + tile_index(I, J) * T.slot_bytes;
    switch (cls) {
    case P64: copy_block<P64, WIDE>(slot, b, T.lo16, ts, lr, lc, i, j0, T.n, L, ldl); break;
    case P32: copy_block<P32, WIDE>(slot, b, T.lo16, ts, lr, lc, i, j0, T.n, L, ldl); break;
    case P16: copy_block<P16, WIDE>(slot, b, T.lo16, ts, lr, lc, i, j0, T.n, L, ldl); break;
    default: copy_block<P8, WIDE>(slot, b, T.lo16, ts, lr, lc, i, j0, T.n, L, ldl); break;
    }
}

// ---------------------------------------------------------------- launchers
static inline int64_t ntiles(const Tiles &T) { return (int64_t)T.nt * (T.nt + 1) / 2; }

// partial: nt (nt + 1) / 2 * (b / 128)^2 doubles
void launch_norms(const Tiles &T, const Source &S, double *partial, double *fro2, double *amax, hipStream_t st)
{
    const int nsub = T.b / 128, parts = nsub == 1 ? 1 : nsub * nsub % 2 ? nsub : nsub * nsub / 2;
    norms_kernel<<<dim3((unsigned)(ntiles(T) * parts)), 1024, 0, st>>>(T, S, parts, partial, fro2, amax);
    if (parts > 1)
        norms_reduce_kernel<<<(unsigned)((ntiles(T) + 255) / 256), 256, 0, st>>>(T.nt, ntiles(T), parts, partial, fro2,
                                                                                 amax);
}

void launch_load(const Tiles &T, const Source &S, hipStream_t st)
{
    load_kernel<<<dim3((unsigned)(T.b / 128 * (T.b / 16)), (unsigned)ntiles(T)), 256, 0, st>>>(T, S);
}

void launch_copy_matrix(const Tiles &T, const double *A, int64_t lda, double *orig, hipStream_t st)
{
    copy_matrix_kernel<<<dim3((unsigned)(T.b / 128 * (T.b / 16)), (unsigned)ntiles(T)), 256, 0, st>>>(T, A, lda, orig);
}

void launch_convert(const Tiles &T, const Panel &P, int k, const uint8_t *qmask, hipStream_t st)
{
    int np = T.nt - k - 1;
    if (np <= 0) return;
    int nsub = T.b / 64;
    convert_kernel<<<dim3(nsub * nsub, np), 256, 0, st>>>(T, P, k, qmask);
}

void launch_logdet(const Tiles &T, double *out, hipStream_t st) { logdet_kernel<<<1, 1024, 0, st>>>(T, out); }

void launch_get_factor(const Tiles &T, double *L, int64_t ldl, hipStream_t st)
{
    const dim3 grid((unsigned)((T.n + 127) / 128), (unsigned)((T.n + 15) / 16));
    if (((uintptr_t)L & 15) == 0 && ldl % 2 == 0) get_factor_kernel<true><<<grid, 256, 0, st>>>(T, L, ldl);
    else get_factor_kernel<false><<<grid, 256, 0, st>>>(T, L, ldl);
}

}  // namespace mpc
