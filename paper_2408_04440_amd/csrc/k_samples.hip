// Covariance from samples: Sigma = scale * Xi Xi^T + nugget I, the estimator
// of the residual covariance (Sec. III.A.3, "Modeling the Temporal Dependence and
// Constructing a Covariance Matrix": the average of the R(T-P) outer products
// of the residual vectors, plus a small diagonal perturbation when there are
// fewer samples than L^2).  A SYRK on the FP64 MFMA with K = the number of samples,
// written straight into the kept FP64 copy in the tile layout (as set_matrix
// does).
#include <algorithm>
#include <mutex>

#include "common.h"
#include "gemm_core.h"
#include "launch.h"

namespace mpc {

// 128 x 128 blocks of Sigma's lower part on the update's core: eight waves of
// 64 x 32 outputs, two workgroups per compute unit.
constexpr int YB = 128, YWM = 2, YWN = 4;
constexpr int YU = 32;       // samples per unit of work (an even number of K slices)
constexpr int YSLOTS = 512;  // workgroups the GPU holds at once
constexpr int YMIN = 4;      // least units a workgroup is started for
typedef CMShape<double, YB, YB, 16, YWM, YWN> YS;

// Where the operands lie: rows of whole blocks and whole units are read from the
// caller's samples; the rows of a last, partial block (edge, YB x m0) and the last,
// partial unit (tail, ldt x YU) from zero-padded copies.
struct Samples {
    const double *x;
    int64_t ldx;
    const double *edge, *tail;
    int64_t ldt;
    int nb, edge_block;  // row blocks; the one in `edge`, or -1
    int units, whole;    // units of K, and those among them read from x
};

// dst[i + k * ldd] = xi[row0 + i + (col0 + k) * ldxi] inside n x m, zero elsewhere.
__global__ __launch_bounds__(256) void pack_samples_kernel(const double *xi, int64_t ldxi, int64_t n, int64_t m,
                                                           int64_t row0, int64_t col0, double *dst, int64_t ldd)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x, k = blockIdx.y;
    if (i >= ldd) return;
    const int64_t r = row0 + i, c = col0 + k;
    dst[i + k * ldd] = (r < n && c < m) ? xi[r + c * ldxi] : 0.0;
}

// Rows of the last tile row (and columns of the last tile) from r0 on: the padding beyond the last row block.
__global__ __launch_bounds__(256) void zero_padding_kernel(Tiles T, int r0, double *orig)
{
    const int J = blockIdx.x, c = blockIdx.y;
    double *col = orig + tile_index(T.nt - 1, J) * (int64_t)T.b * T.b + (int64_t)c * T.b;
    for (int r = ((J == T.nt - 1 && c >= r0) ? 0 : r0) + threadIdx.x; r < T.b; r += 256) col[r] = 0.0;
}

// orig = scale * acc (+ nugget on the diagonal below n) for block (bi, bj), and
// its mirror image where that lies in the same (diagonal) tile.
__device__ inline void write_cov(const Tiles &T, int bi, int bj, const double4_t (&acc)[YS::MB][YS::NB], double scale,
                                 double nugget, double *orig)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = wave % YWM, wn = wave / YWM, gi = lane & 15, gg = lane >> 4;
    const int b = T.b, per = b / YB, I = bi / per, J = bj / per, tm = bi % per, tn = bj % per;
    double *dst = orig + tile_index(I, J) * (int64_t)b * b;
#pragma unroll
    for (int m = 0; m < YS::MB; ++m)
#pragma unroll
        for (int q = 0; q < YS::NB; ++q) {
            const int r = tm * YB + wm * (YB / YWM) + m * 16 + gi;  // swapped operands: lane gi owns row r
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int c = tn * YB + wn * (YB / YWN) + q * 16 + acc_row<double>(gg, v);
                double val = scale * acc[m][q][v];
                if (I == J && r == c && (int64_t)I * b + r < T.n) val += nugget;
                dst[r + (int64_t)c * b] = val;
                if (I == J && bi != bj) dst[c + (int64_t)r * b] = val;
            }
        }
}

// Work item of the products: blocks [0, full) are taken whole, one workgroup each;
// the units of the others are dealt out evenly, in one run, to the remaining
// workgroups.  A run ends inside a block, so most of these hold two or three
// pieces; every piece goes to its own place in `part` and syrk_finish_kernel adds
// them in order.
struct Deal {
    int full, rest, wgs;  // whole blocks, dealt blocks, workgroups of the dealt ones
    __host__ __device__ int64_t begin(int w, int units) const { return (int64_t)rest * units * w / wgs; }
};

// What bounds it: the FP64 MFMA.  (N = 4,900, 6000 samples: 3.46 -> 2.77 ms and
// 0.04 to add the pieces, 58 TFLOP/s of the lower part.  With whole blocks alone the
// last round of workgroups was half empty, 780 blocks on 512 places; both halves of
// the diagonal tiles were computed, and the samples were first copied whole into a
// padded buffer allocated for the call, another 0.5 ms.)
__global__ __launch_bounds__(YS::NTH) __attribute__((amdgpu_waves_per_eu(4))) void syrk_samples_kernel(
    Tiles T, Samples P, Deal D, double scale, double nugget, double *orig, double *part)
{
    extern __shared__ __align__(16) char smem_raw[];
    double4_t acc[YS::MB][YS::NB];
    int64_t u, ue;
    int w = -1;
    if ((int)blockIdx.x < D.full) {
        u = xcd_remap(blockIdx.x, D.full) * P.units;
        ue = u + P.units;
    } else {
        w = (int)xcd_remap(blockIdx.x - D.full, D.wgs);
        u = (int64_t)D.full * P.units + D.begin(w, P.units);
        ue = (int64_t)D.full * P.units + D.begin(w + 1, P.units);
    }
#pragma unroll 1
    while (u < ue) {
        const int64_t blk = u / P.units;
        const int u0 = (int)(u - blk * P.units), u1 = (int)min(ue - blk * P.units, (int64_t)P.units);
        int bi, bj;
        tile_ij(blk, bi, bj);
#pragma unroll
        for (int m = 0; m < YS::MB; ++m)
#pragma unroll
            for (int q = 0; q < YS::NB; ++q) acc[m][q] = (double4_t){0.0, 0.0, 0.0, 0.0};
        const bool ea = bi == P.edge_block, eb = bj == P.edge_block;
        const double *A = ea ? P.edge : P.x + (int64_t)bi * YB, *B = eb ? P.edge : P.x + (int64_t)bj * YB;
        int64_t lda = ea ? YB : P.ldx, ldb = eb ? YB : P.ldx;
        // offsets within one call of the core are 32-bit
        const int most = (int)min((int64_t)(0x7FFFFFFF / YU) / P.ldx, (int64_t)(1 << 20));
        int k = u0;
#pragma unroll 1
        while (k < u1) {
            const bool t = k >= P.whole;
            const int e = t ? u1 : min(min(u1, P.whole), k + most);
            const double *a = t ? P.tail + (int64_t)bi * YB : A + (int64_t)k * YU * lda;
            const double *bb = t ? P.tail + (int64_t)bj * YB : B + (int64_t)k * YU * ldb;
            cm_block_deep<double, YB, YB, 16, YWM, YWN, true>(a, t ? P.ldt : lda, bb, t ? P.ldt : ldb, (e - k) * YU, acc,
                                                              (double *)smem_raw);
            k = e;
        }
        if (w < 0) {
            write_cov(T, bi, bj, acc, scale, nugget, orig);
        } else {
            // pieces before this one: one per workgroup before w and one more per
            // block boundary before u
            double *dst = part + ((int64_t)w + blk - D.full) * YB * YB + threadIdx.x;
#pragma unroll
            for (int m = 0; m < YS::MB; ++m)
#pragma unroll
                for (int q = 0; q < YS::NB; ++q)
#pragma unroll
                    for (int v = 0; v < 4; ++v) dst[((m * YS::NB + q) * 4 + v) * YS::NTH] = acc[m][q][v];
        }
        u += u1 - u0;
    }
}

// Dealt block full + blockIdx.x: its pieces, added in the order of their samples.
__global__ __launch_bounds__(YS::NTH) void syrk_finish_kernel(Tiles T, Samples P, Deal D, double scale, double nugget,
                                                              double *orig, const double *part)
{
    const int64_t u0 = (int64_t)blockIdx.x * P.units, u1 = u0 + P.units;
    // first workgroup whose run reaches past u0
    int w = (int)(u0 * D.wgs / ((int64_t)D.rest * P.units));
    while (w > 0 && D.begin(w, P.units) > u0) --w;
    while (D.begin(w + 1, P.units) <= u0) ++w;
    double4_t acc[YS::MB][YS::NB];
#pragma unroll
    for (int m = 0; m < YS::MB; ++m)
#pragma unroll
        for (int q = 0; q < YS::NB; ++q) acc[m][q] = (double4_t){0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
    for (; w < D.wgs && D.begin(w, P.units) < u1; ++w) {
        if (D.begin(w + 1, P.units) == D.begin(w, P.units)) continue;
        const double *src = part + ((int64_t)w + blockIdx.x) * YB * YB + threadIdx.x;
#pragma unroll
        for (int m = 0; m < YS::MB; ++m)
#pragma unroll
            for (int q = 0; q < YS::NB; ++q)
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[m][q][v] += src[((m * YS::NB + q) * 4 + v) * YS::NTH];
    }
    int bi, bj;
    tile_ij(D.full + blockIdx.x, bi, bj);
    write_cov(T, bi, bj, acc, scale, nugget, orig);
}

// Read in place where the core's 16-byte loads allow it (an aligned base, an even
// leading dimension, offsets of one unit within 32 bits); packed whole otherwise.
static bool samples_in_place(const double *xi, int64_t ldxi)
{
    return ((uintptr_t)xi & 15) == 0 && ldxi % 2 == 0 && ldxi <= 0x7FFFFFFF / (2 * YU);
}

static Samples samples_shape(const Tiles &T, const double *xi, int64_t ldxi, int64_t m)
{
    Samples P = {};
    P.nb = (int)((T.n + YB - 1) / YB);
    P.units = (int)((m + YU - 1) / YU);
    P.ldt = (int64_t)P.nb * YB;
    const bool in = samples_in_place(xi, ldxi);
    P.ldx = in ? ldxi : P.ldt;
    P.x = in ? xi : nullptr;
    P.whole = in ? (int)(m / YU) : P.units;
    P.edge_block = (in && T.n % YB != 0) ? P.nb - 1 : -1;
    return P;
}

// As many whole blocks as fill the GPU's places evenly; the rest dealt out over all places.
static Deal samples_deal(const Samples &P)
{
    const int blocks = P.nb * (P.nb + 1) / 2;
    Deal D;
    D.full = blocks / YSLOTS * YSLOTS;
    D.rest = blocks - D.full;
    D.wgs = D.rest ? (int)std::min<int64_t>(YSLOTS, ((int64_t)D.rest * P.units + YMIN - 1) / YMIN) : 0;
    return D;
}

// Doubles of scratch: the padded copies and the pieces of dealt blocks.
int64_t cov_samples_scratch(const Tiles &T, const double *xi, int64_t ldxi, int64_t m)
{
    const Samples P = samples_shape(T, xi, ldxi, m);
    const Deal D = samples_deal(P);
    const int64_t copies = P.x ? (P.edge_block >= 0 ? (int64_t)P.whole * YU * YB : 0) + (P.whole < P.units ? P.ldt * YU : 0)
                               : P.ldt * P.units * YU;
    return copies + (D.rest ? (int64_t)(D.wgs + D.rest) * YB * YB : 0);
}

static void pack(const double *xi, int64_t ldxi, int64_t n, int64_t m, int64_t row0, int64_t col0, double *dst,
                 int64_t ldd, int64_t cols, hipStream_t st)
{
    for (int64_t c = 0; c < cols; c += 65535)
        pack_samples_kernel<<<dim3((unsigned)((ldd + 255) / 256), (unsigned)std::min<int64_t>(65535, cols - c)), 256, 0, st>>>(
            xi, ldxi, n, m, row0, col0 + c, dst + c * ldd, ldd);
}

int launch_cov_samples(const Tiles &T, const double *xi, int64_t ldxi, int64_t m, double scale, double nugget,
                       double *scratch, double *orig, hipStream_t st)
{
    Samples P = samples_shape(T, xi, ldxi, m);
    const Deal D = samples_deal(P);
    if (!P.x) {
        pack(xi, ldxi, T.n, m, 0, 0, scratch, P.ldt, (int64_t)P.units * YU, st);
        P.x = scratch;
        scratch += P.ldt * P.units * YU;
    } else {
        if (P.edge_block >= 0) {
            pack(xi, ldxi, T.n, m, (int64_t)P.edge_block * YB, 0, scratch, YB, (int64_t)P.whole * YU, st);
            P.edge = scratch;
            scratch += (int64_t)P.whole * YU * YB;
        }
        if (P.whole < P.units) {
            pack(xi, ldxi, T.n, m, 0, (int64_t)P.whole * YU, scratch, P.ldt, YU, st);
            P.tail = scratch;
            scratch += P.ldt * YU;
        }
    }
    const int r0 = P.nb * YB - (T.nt - 1) * T.b;
    if (r0 < T.b) zero_padding_kernel<<<dim3((unsigned)T.nt, (unsigned)T.b), 256, 0, st>>>(T, r0, orig);
    static std::once_flag attr;
    std::call_once(attr, [] {
        (void)hipFuncSetAttribute((const void *)syrk_samples_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                  (int)YS::SMEM);
    });
    syrk_samples_kernel<<<(unsigned)(D.full + D.wgs), YS::NTH, YS::SMEM, st>>>(T, P, D, scale, nugget, orig, scratch);
    if (D.rest) syrk_finish_kernel<<<(unsigned)D.rest, YS::NTH, 0, st>>>(T, P, D, scale, nugget, orig, scratch);
    return 0;
}

}  // namespace mpc
