// The factorization's tasks (Sec. V.A): POTRF of a diagonal tile, TRSM of the
// panel below it, and the SYRK/GEMM trailing update grouped per precision
// class, all for gfx950.
#include "common.h"
#include "gemm_core.h"
#include "launch.h"

namespace mpc {

// ---------------------------------------------------------------- blocks of 64 in LDS
// Shared by the diagonal tile's POTRF and the panel TRSM: four waves, each
// owning 16 rows; 64 x 64 blocks in LDS column-major with leading dimension LD64.
constexpr int LD64 = 66;

// orders one wavefront's LDS accesses across lanes (the hardware executes a
// wave's LDS instructions in order; this keeps the compiler from moving them)
__device__ inline void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Lane N of every row of 16 lanes, to the whole row (a DPP move).
template <int N> __device__ inline double row_bcast(double v)
{
    return __longlong_as_double(__builtin_amdgcn_update_dpp(0ll, __double_as_longlong(v), 0x150 + N, 0xf, 0xf, true));
}

// t[j] -= m * (lane j of the row of 16's s) for j = C + 1 .. 15: one DPP
// multiply-add each (5 cycles; the compiler makes a move and a multiply-add of
// it, 12 cycles, and gathers the moves of many columns until they spill).  The
// s_nops cover the wait states between a VALU write and a DPP read of it, s at
// the start and the last t at the end, which the compiler does not see here.
#define MPC_U(j) "\n\tv_fmac_f64_dpp %" #j ", -%[s], %[m] row_newbcast:" #j " row_mask:0xf bank_mask:0xf"
#define MPC_FROM_15 MPC_U(15)
#define MPC_FROM_14 MPC_U(14) MPC_FROM_15
#define MPC_FROM_13 MPC_U(13) MPC_FROM_14
#define MPC_FROM_12 MPC_U(12) MPC_FROM_13
#define MPC_FROM_11 MPC_U(11) MPC_FROM_12
#define MPC_FROM_10 MPC_U(10) MPC_FROM_11
#define MPC_FROM_9 MPC_U(9) MPC_FROM_10
#define MPC_FROM_8 MPC_U(8) MPC_FROM_9
#define MPC_FROM_7 MPC_U(7) MPC_FROM_8
#define MPC_FROM_6 MPC_U(6) MPC_FROM_7
#define MPC_FROM_5 MPC_U(5) MPC_FROM_6
#define MPC_FROM_4 MPC_U(4) MPC_FROM_5
#define MPC_FROM_3 MPC_U(3) MPC_FROM_4
#define MPC_FROM_2 MPC_U(2) MPC_FROM_3
#define MPC_FROM_1 MPC_U(1) MPC_FROM_2
#define MPC_ROW_ASM(body)                                                                                             \
    asm("s_nop 1" body "\n\ts_nop 1"                                                                                  \
        : "+v"(t[0]), "+v"(t[1]), "+v"(t[2]), "+v"(t[3]), "+v"(t[4]), "+v"(t[5]), "+v"(t[6]), "+v"(t[7]),             \
          "+v"(t[8]), "+v"(t[9]), "+v"(t[10]), "+v"(t[11]), "+v"(t[12]), "+v"(t[13]), "+v"(t[14]), "+v"(t[15])        \
        : [s] "v"(s), [m] "v"(m))
template <int C> __device__ inline void row_update(double (&t)[16], double s, double m)
{
    if constexpr (C == 0) MPC_ROW_ASM(MPC_FROM_1);
    else if constexpr (C == 1) MPC_ROW_ASM(MPC_FROM_2);
    else if constexpr (C == 2) MPC_ROW_ASM(MPC_FROM_3);
    else if constexpr (C == 3) MPC_ROW_ASM(MPC_FROM_4);
    else if constexpr (C == 4) MPC_ROW_ASM(MPC_FROM_5);
    else if constexpr (C == 5) MPC_ROW_ASM(MPC_FROM_6);
    else if constexpr (C == 6) MPC_ROW_ASM(MPC_FROM_7);
    else if constexpr (C == 7) MPC_ROW_ASM(MPC_FROM_8);
    else if constexpr (C == 8) MPC_ROW_ASM(MPC_FROM_9);
    else if constexpr (C == 9) MPC_ROW_ASM(MPC_FROM_10);
    else if constexpr (C == 10) MPC_ROW_ASM(MPC_FROM_11);
    else if constexpr (C == 11) MPC_ROW_ASM(MPC_FROM_12);
    else if constexpr (C == 12) MPC_ROW_ASM(MPC_FROM_13);
    else if constexpr (C == 13) MPC_ROW_ASM(MPC_FROM_14);
    else if constexpr (C == 14) MPC_ROW_ASM(MPC_FROM_15);
}

// A diagonal element d of L as the substitutions divide by it: 0 in place of infinity
// (an infinite entry of the matrix).  With r = 1 / d = 0 div_by then gives 0, as
// x / d does; with d itself its remainder would be 0 * infinity.
__device__ inline double as_divisor(double d) { return d == __builtin_inf() ? 0.0 : d; }

// s = sqrt(d) and r = 1 / s to about 47 bits, for d in [2^-900, 2^900]: one
// step of Goldschmidt's iteration from the hardware's estimate, the root then
// corrected by its exact remainder (a perfect square gives its root exactly).
__device__ inline void sqrt_rcp(double d, double &s, double &r)
{
    const double y = __builtin_amdgcn_rsq(d);
    double g = d * y, h = 0.5 * y;
    const double e = __builtin_fma(-h, g, 0.5);
    g = __builtin_fma(g, e, g);
    h = __builtin_fma(h, e, h);
    s = __builtin_fma(__builtin_fma(-g, g, d), h, g);
    r = h + h;
}

// acc[ct] += X(rows 16w.., k) Y(rows 16ct.., k)^T over columns k0 .. k1 - 1 (a
// multiple of 16) of the LDS blocks.  Operands swapped: a lane holds row gi of its wave's 16 and
// columns gg + 4v of each 16-column tile.
__device__ inline void mma64(double4_t (&acc)[4], const double *X, const double *Y, int wave, int gi, int gg,
                             int k0 = 0, int k1 = 64)
{
    struct Ops {
        double x[2], y[2][4];
    } u, w;
    auto load = [&](int k, Ops &o) {
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int row = (k + 4 * s + gg) * LD64 + gi;
            o.x[s] = X[row + wave * 16];
#pragma unroll
            for (int ct = 0; ct < 4; ++ct) o.y[s][ct] = Y[row + ct * 16];
        }
    };
    auto mma = [&](const Ops &o) {
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int ct = 0; ct < 4; ++ct)
                acc[ct] = __builtin_amdgcn_mfma_f64_16x16x4f64(o.y[s][ct], o.x[s], acc[ct], 0, 0, 0);
    };
    load(k0, u);
#pragma unroll 1
    for (int k = k0; k < k1; k += 16) {  // the next eight columns are read while eight are multiplied
        load(k + 8, w);
        mma(u);
        if (k + 16 < k1) load(k + 16, u);
        mma(w);
    }
}

// v = a block of the matrix less products: those of 64 columns are summed from zero
// and added once, so that v is rounded at its size once per 64 columns, not once per
// product, and the error does not grow with the tile (1024: 6 to 2 u).
__device__ inline void zero64(double4_t (&v)[4])
{
#pragma unroll
    for (int ct = 0; ct < 4; ++ct) v[ct] = (double4_t){0.0, 0.0, 0.0, 0.0};
}
__device__ inline void add64(double4_t (&v)[4], const double4_t (&sum)[4])
{
#pragma unroll
    for (int ct = 0; ct < 4; ++ct) v[ct] += sum[ct];
}

// Panel p of X = -acc L^-T for a wave's 16 rows: L the lower 64 x 64 block in
// LDS (its columns 16 p .. 16 p + 15 are read), d = L(16 p + gi, 16 p + gi) as
// as_divisor gives it, rl = 1 / L(16 p + gi, 16 p + gi),
// acc the negated 16 x 64 right-hand side, acc[0] the current 16 columns: the
// later panels' sums move up by one, so that the four panels share one copy of
// the code (a diagonal workgroup runs it once, and four copies cost more in
// instruction fetches than the moves).  Every lane gathers its row of the panel
// (the four lane groups hold the same rows) and substitutes column by column
// against broadcasts of the diagonal block's rows from other lanes; the
// panel's product with the rest of L goes to the later sums on the MFMA.
// put(t, v): lane (gi, gg) delivers X(gi, 16 p + 4 t + gg).
template <typename Put>
__device__ inline void wave_trsm16(double4_t (&acc)[4], int p, const double *L, double d, double rl, double *scratch,
                                   int gi, int gg, Put put)
{
    const double *Lp = L + 16 * p * LD64 + 16 * p + gi;
    double x[16], ld[16];  // lane gi: its row, and row gi of the panel's 16 x 16 diagonal block
    wave_sync();
#pragma unroll
    for (int v = 0; v < 4; ++v) scratch[gi * 17 + gg + 4 * v] = -acc[0][v];
#pragma unroll
    for (int c = 0; c < 16; ++c) ld[c] = Lp[c * LD64];
    wave_sync();
#pragma unroll
    for (int c = 0; c < 16; ++c) x[c] = scratch[gi * 17 + c];
    static_for<0, 16>([&](auto C) {
        constexpr int c = C;
        x[c] = div_by(x[c], row_bcast<c>(d), row_bcast<c>(rl));
        row_update<c>(x, ld[c], x[c]);
    });
    double a[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const double x0 = x[4 * t], x1 = x[4 * t + 1], x2 = x[4 * t + 2], x3 = x[4 * t + 3];
        const double lo = gg & 1 ? x1 : x0, hi = gg & 1 ? x3 : x2;
        a[t] = gg & 2 ? hi : lo;  // x[4 t + gg]
        put(t, a[t]);
    }
#pragma unroll
    for (int r = 1; r < 4; ++r) {
        double4_t sum = {0.0, 0.0, 0.0, 0.0};  // added once, as in add64
        if (p + r < 4) {
#pragma unroll
            for (int t = 0; t < 4; ++t)
                sum = __builtin_amdgcn_mfma_f64_16x16x4f64(Lp[(4 * t + gg) * LD64 + 16 * r], a[t], sum, 0, 0, 0);
        }
        acc[r - 1] = acc[r] + sum;
    }
}

// Columns h .. h + 15 of the block S by one wave, right-looking in LDS, with the
// library's square root and division: for pivots outside the range of sqrt_rcp,
// among them zero, negative, infinite and NaN.
__device__ __attribute__((noinline)) void panel_potrf16(double *S, int h, int lane, int64_t col0, int64_t n,
                                                        unsigned long long *info)
{
#pragma unroll 1
    for (int c = h; c < h + 16; ++c) {
        wave_sync();
        const double d = S[c * LD64 + c], x = S[c * LD64 + lane];
        if (lane == 0 && !(d > 0.0) && col0 + c < n) atomicMin(info, (unsigned long long)(col0 + c + 1));
        const double piv = sqrt(d), l = lane == c ? piv : x / piv;
        wave_sync();
        S[c * LD64 + lane] = lane >= c ? l : 0.0;
        wave_sync();
#pragma unroll 1
        for (int j = c + 1; j < h + 16; ++j) S[j * LD64 + lane] -= l * S[c * LD64 + j];
    }
}

// Cholesky of the lower 64 x 64 block S in LDS by four waves, in panels of 16
// columns: one wave factors the panel, lane r holding row r, with the panel's
// diagonal block held once more by every row of 16 lanes for the broadcasts; the
// later tiles are updated on the MFMA.  Zeros go
// above the diagonal.  out(p) runs in every thread once panel p is in LDS,
// done(p) in every thread after a barrier behind it.  A pivot that is not positive (or NaN) records its
// 1-based global column col0 + c + 1 in *info (minimum over failures); the
// computation then continues on NaNs and still terminates.
template <typename Out, typename Done>
__device__ inline void block_potrf64(double *S, int wave, int lane, int64_t col0, int64_t n, unsigned long long *info,
                                     Out out, Done done)
{
    const int gi = lane & 15, gg = lane >> 4;
#pragma unroll 1
    for (int p = 0; p < 4; ++p) {
        const int h = 16 * p;
        if (wave == 0) {
            double x[16], xd[16];  // row `lane`, and row h + gi: every 16 lanes hold the diagonal block to broadcast
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                xd[j] = S[(h + j) * LD64 + h + gi];
                x[j] = S[(h + j) * LD64 + lane];
            }
            bool ordinary = true;  // every pivot in [2^-900, 2^900)
            static_for<0, 16>([&](auto C) {
                constexpr int c = C;
                const double d = row_bcast<c>(xd[c]);
                ordinary = ordinary && (uint32_t)(__double_as_longlong(d) >> 32) - 0x07B00000u < 0x78300000u - 0x07B00000u;
                double piv, r;
                sqrt_rcp(d, piv, r);
                xd[c] = div_by(xd[c], piv, r);
                if (gi == c) xd[c] = piv;
                x[c] = div_by(x[c], piv, r);
                if (lane == h + c) x[c] = piv;
                row_update<c>(xd, xd[c], xd[c]);
                row_update<c>(x, xd[c], x[c]);
            });
            if (__builtin_expect(__ballot(ordinary) == ~0ull, 1)) {
#pragma unroll
                for (int j = 0; j < 16; ++j) S[(h + j) * LD64 + lane] = lane >= h + j ? x[j] : 0.0;
            } else {
                panel_potrf16(S, h, lane, col0, n, info);
            }
        }
        __syncthreads();
        out(p);
        // lower tiles (rt, ct) of the trailing 64 - h - 16 columns, dealt to the waves
        const int q = 3 - p;
        for (int t = wave; t < q * (q + 1) / 2; t += 4) {
            const int i = t < 1 ? 0 : t < 3 ? 1 : 2, j = t - i * (i + 1) / 2;
            const int rt = p + 1 + i, ct = p + 1 + j;
            double4_t a = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const double *col = S + (h + 4 * s + gg) * LD64 + gi;
                a = __builtin_amdgcn_mfma_f64_16x16x4f64(col[ct * 16], col[rt * 16], a, 0, 0, 0);
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) S[(ct * 16 + gg + 4 * v) * LD64 + rt * 16 + gi] -= a[v];
        }
        stores_done();
        __syncthreads();
        done(p);
    }
}

// ---------------------------------------------------------------- POTRF of a diagonal tile
// One launch for the whole b x b tile (b = 64 nb), blocks of 64.  What bounds it
// is the chain of nb diagonal blocks: factor the block, solve the one below it,
// update the next.  A launch each for a block's factor, the rows below it and their
// update cost about 60 us a block, one launch 18 us, and 16 us since panels of 16
// columns are handed on as they are factored (a 1024 tile: 0.96 -> 0.25 ms).
// Every block has its workgroup, which sums its products with the blocks to its
// left as these become known and waits for the rest of its turn in place:
//   diagonal workgroup m: blocks (m, m-1) and (m, m) -- the solve of the first
//       feeds the second without leaving the compute unit, so the chain crosses
//       memory once per block;
//   workgroup (i, m), i >= m + 2: block (i, m).
// prog[i] counts the finished 16-column panels of block row i: blocks finish in
// column order, four panels at a time, a diagonal block panel by panel, so that
// the rows below solve against a panel while the next one is factored.  Finished blocks
// are written and read with device-scope accesses, and their stores have
// completed before the count is raised.  Places are given out by a ticket
// counter in column order, and every block depends on blocks with earlier
// tickets only, so the earliest workgroup can always finish.  A wait that lasts
// longer than WAIT_TICKS sets *info to 0, which the host reports as an error.
__device__ inline double ld_dev(const double *p)
{
    return __longlong_as_double(
        (long long)__hip_atomic_load((const unsigned long long *)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}
__device__ inline void st_dev(double *p, double v)
{
    __hip_atomic_store((unsigned long long *)p, (unsigned long long)__double_as_longlong(v), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}

// One thread: until prog[i] >= vi and prog[m] >= vm; false if the wait ran out.
__device__ inline bool wait_prog(const int *prog, int i, int vi, int m, int vm, unsigned long long *info)
{
    const long long t0 = wall_clock64();
    for (unsigned k = 1;; ++k) {
        const int a = __hip_atomic_load(prog + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const int c = __hip_atomic_load(prog + m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (a >= vi && c >= vm) return true;
        __builtin_amdgcn_s_sleep(1);
        if ((k & 255) == 0 && (__hip_atomic_load(info, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0 ||
                               wall_clock64() - t0 > WAIT_TICKS)) {
            atomicMin(info, 0ull);
            return false;
        }
    }
}

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void potrf_tile_kernel(
    double *tile, int b, int64_t col0, int64_t n, int *ctl, unsigned long long *info, unsigned long long *pmax, int npmax)
{
    __builtin_amdgcn_s_setprio(3);  // the panel chain: issue ahead of update waves sharing the SIMD
    __shared__ double A[64 * LD64], Bs[64 * LD64];
    __shared__ double scratch[4][16 * 17];
    __shared__ int s_word;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, gi = lane & 15, gg = lane >> 4;
    const int nb = b / 64;
    int *prog = ctl + 1;
    if (blockIdx.x == 0)  // the panel's maxima, which its TRSM collects after this launch
        for (int q = tid; q < npmax; q += 256) pmax[q] = 0;
    if (tid == 0) s_word = atomicAdd(ctl, 1);
    __syncthreads();
    int m = 0, i = __builtin_amdgcn_readfirstlane(s_word);  // column order: diagonal m, then (i, m) for i = m + 2 .. nb - 1
    for (;; ++m) {
        const int cnt = 1 + max(0, nb - 2 - m);
        if (i < cnt) break;
        i -= cnt;
    }
    const bool diag = i == 0;
    i = diag ? m : m + 1 + i;
    const int ca = diag ? m - 1 : m;  // column of the block solved here (none for m = 0 on the diagonal)
    __syncthreads();

    // block (r, c); within a block a uniform column base plus a lane's 32-bit byte offset
    const int64_t cs = (int64_t)b * 8;
    auto at = [&](int r, int c) { return (char *)tile + (int64_t)(64 * r) * 8 + 64 * c * cs; };
    const uint32_t own8 = (wave * 16 + gi + gg * b) * 8, lin8 = (lane + wave * b) * 8;
    // the blocks themselves start the sums, negated; the mirrored block above the diagonal becomes zero
    double4_t acc1[4], acc2[4], sum[4];
    zero64(acc1);
    zero64(acc2);
    if (ca >= 0) {
#pragma unroll
        for (int q = 0; q < 16; ++q) acc1[q / 4][q % 4] = -*(const double *)(at(i, ca) + 4 * q * cs + own8);
    }
    if (diag) {
#pragma unroll
        for (int q = 0; q < 16; ++q) acc2[q / 4][q % 4] = -*(const double *)(at(i, i) + 4 * q * cs + own8);
    }
    if (ca >= 0) {
        char *up = at(ca, i);
        for (int q = 0; q < 16; ++q) *(double *)(up + 4 * q * cs + lin8) = 0.0;
    }

    double ra[16], rb[16];
    auto load = [&](int j) {
        const char *pa = at(i, j), *pb = at(ca, j);
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            ra[q] = ld_dev((const double *)(pa + 4 * q * cs + lin8));
            rb[q] = ld_dev((const double *)(pb + 4 * q * cs + lin8));
        }
    };
    int have = 0;
    for (int j = 0; j < ca; ++j) {
        if (j >= have) {
            if (tid == 0) {
                int ok = wait_prog(prog, i, 4 * j + 4, ca, 4 * j + 4, info);
                if (ok) ok = min(__hip_atomic_load(prog + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT),
                                 __hip_atomic_load(prog + ca, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) / 4;
                s_word = ok;
            }
            __syncthreads();
            have = s_word;
            if (have == 0) return;
            load(j);
        }
        __syncthreads();  // the previous products have been read from LDS
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            A[(wave + 4 * q) * LD64 + lane] = ra[q];
            Bs[(wave + 4 * q) * LD64 + lane] = rb[q];
        }
        __syncthreads();
        if (j + 1 < ca && j + 1 < have) load(j + 1);
        zero64(sum);
        mma64(sum, A, Bs, wave, gi, gg);
        add64(acc1, sum);
        if (diag) {
            zero64(sum);
            mma64(sum, A, A, wave, gi, gg);
            add64(acc2, sum);
        }
    }

    if (ca >= 0) {
        const char *pl = at(ca, ca);
        char *px = at(i, ca);
        __syncthreads();  // the last products have been read from LDS
        zero64(sum);
#pragma unroll 1
        for (int p = 0; p < 4; ++p) {  // panel p of L(ca, ca) into Bs, then this block's panel
            if (tid == 0) s_word = wait_prog(prog, ca, 4 * ca + p + 1, ca, 4 * ca + p + 1, info);
            __syncthreads();
            if (!s_word) return;
            const double d = ld_dev((const double *)(pl + 16 * p * (8 + cs) + (uint32_t)((gi + gi * b) * 8)));
            double l[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) l[q] = ld_dev((const double *)(pl + (16 * p + 4 * q) * cs + lin8));
#pragma unroll
            for (int q = 0; q < 4; ++q) Bs[(16 * p + wave + 4 * q) * LD64 + lane] = l[q];
            const double rl = 1.0 / d;
            __syncthreads();
            wave_trsm16(acc1, p, Bs, as_divisor(d), rl, scratch[wave], gi, gg, [&](int t, double v) {
                st_dev((double *)(px + (16 * p + 4 * t) * cs + own8), v);
                if (diag) A[(16 * p + 4 * t + gg) * LD64 + wave * 16 + gi] = v;
            });
            if (diag) {
                __syncthreads();
                mma64(sum, A, A, wave, gi, gg, 16 * p, 16 * p + 16);
            }
        }
        if (diag) add64(acc2, sum);
        stores_done();
        __syncthreads();
        if (tid == 0) __hip_atomic_store(prog + i, 4 * ca + 4, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (!diag) return;
    // the diagonal block: Bs is free, every wave is past its solve
#pragma unroll
    for (int ct = 0; ct < 4; ++ct)
#pragma unroll
        for (int v = 0; v < 4; ++v) Bs[(ct * 16 + gg + 4 * v) * LD64 + wave * 16 + gi] = -acc2[ct][v];
    __syncthreads();
    char *pd = at(m, m);
    block_potrf64(
        Bs, wave, lane, col0 + 64 * (int64_t)m, n, info,
        [&](int p) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
                st_dev((double *)(pd + (16 * p + 4 * q) * cs + lin8), Bs[(16 * p + wave + 4 * q) * LD64 + lane]);
        },
        [&](int p) {
            if (tid == 0) __hip_atomic_store(prog + m, 4 * m + p + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        });
}

// Words of control memory per diagonal tile: the ticket and the block rows'
// counts; all zero before the tile's launch.
int potrf_ctl_words(int b) { return 1 + b / 64; }

void launch_potrf_tile(const Tiles &T, const Panel &P, int k, int *ctl, hipStream_t st)
{
    const int b = T.b, nb = b / 64;
    double *tile = (double *)(T.slots + tile_index(k, k) * T.slot_bytes);
    const int off = (nb - 1) * (nb - 2) / 2;  // blocks two or more below the diagonal
    potrf_tile_kernel<<<nb + off, 256, 0, st>>>(tile, b, (int64_t)k * b, T.n,
                                                ctl + (int64_t)k * potrf_ctl_words(b), P.info, P.pmax, T.nt);
}

// ---------------------------------------------------------------- TRSM
// The panel of step k: X = W L^-T for 64-row strips of the tiles I > k, W the
// work tile (FP64, or FP32 for lower classes), X = p64[I].  Four waves, each
// its own 16 rows from end to end: column blocks of 64, whose product with the
// solved columns runs on the FP64 MFMA straight from registers (X and L, three
// chunks of 16 columns in flight, no barrier), then the substitution of
// wave_trsm16; the waves only share the diagonal block in LDS.  What bounds a
// strip is its b / 64 column blocks in sequence, what bounds many strips the
// MFMA (248 strips of 512 columns: 0.33 -> 0.15 ms, where the products alone take
// 0.055 ms on their compute unit).  The strip's largest |X| is folded into pmax[I] (atomic max of the FP64
// bits, which order like the values; the tile's POTRF zeroes pmax), and the first
// column holding an Inf or NaN into P.info (every off-diagonal factor tile
// passes here, so a non-finite value is reported even where a low-precision
// code would saturate it).  An FP64 tile whose only consumers are FP64 updates
// is stored from here as well and needs no conversion.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void trsm_kernel(Tiles T, Panel P, int k, const double *__restrict__ L,
                                                                                            const uint8_t *qmask)
{
    __builtin_amdgcn_s_setprio(3);  // the panel chain: issue ahead of update waves sharing the SIMD
    __shared__ double Ls[64 * LD64];
    __shared__ double dia[64], inv[64], scratch[4][16 * 17];
    const int b = T.b, I = k + 1 + blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, gi = lane & 15, gg = lane >> 4;
    const bool wf32 = T.map[I + (int64_t)k * T.nt] != P64;
    const bool direct = panel_direct(T.map[I + (int64_t)k * T.nt], qmask[I]);  // the stored tile and its only copy are X
    // addresses: a uniform column base plus a lane's 32-bit byte offset
    const int row0 = blockIdx.x * 64;
    char *W = T.slots + tile_index(I, k) * T.slot_bytes + (int64_t)row0 * (wf32 ? 4 : 8);
    char *X = (char *)(P.p64 + (int64_t)I * b * b + row0);
    const char *Lc = (const char *)L;
    const uint32_t own = wave * 16 + gi + gg * b;  // row gi of the wave, column gg
    const uint32_t own8 = own * 8, own4 = own * 4, lop8 = (gi + gg * b) * 8, dia8 = (lane + wave * b) * 8;
    const int64_t cs = (int64_t)b * 8;  // bytes from column to column
    double xmax = 0.0;     // largest |X| of this lane's row
    int bad = 0x7FFFFFFF;  // first column (in the tile) of a non-finite X
    double lv[16], dv;     // the next diagonal block and its diagonal, read ahead
    auto load_diag = [&](int cb) {
        dv = *(const double *)(Lc + (int64_t)cb * 8 + cb * cs + (lane + lane * b) * 8);
#pragma unroll
        for (int q = 0; q < 16; ++q) lv[q] = *(const double *)(Lc + (int64_t)cb * 8 + (cb + 4 * q) * cs + dia8);
    };
    load_diag(0);
    for (int cb = 0; cb < b; cb += 64) {
#pragma unroll
        for (int q = 0; q < 16; ++q) Ls[(wave + 4 * q) * LD64 + lane] = lv[q];
        if (wave == 0) {
            dia[lane] = as_divisor(dv);
            inv[lane] = 1.0 / dv;
        }
        // right-hand side, read ahead of the products
        double4_t w[4], acc[4];
        if (wf32) {
#pragma unroll
            for (int q = 0; q < 16; ++q)
                w[q / 4][q % 4] = (double)*(const float *)(W + (cb + 4 * q) * (cs / 2) + own4);
        } else {
#pragma unroll
            for (int q = 0; q < 16; ++q) w[q / 4][q % 4] = *(const double *)(W + (cb + 4 * q) * cs + own8);
        }
#pragma unroll
        for (int ct = 0; ct < 4; ++ct) acc[ct] = (double4_t){0.0, 0.0, 0.0, 0.0};
        // MFMA step s of a chunk: columns 8 kc + 4 s + gg of X and L
        struct Chunk {
            double a[2], l[2][4];
        } c0, c1, c2, c3;
        auto load = [&](int kc, Chunk &c) {
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const int64_t o = (kc * 8 + 4 * s) * cs;
                c.a[s] = *(const double *)(X + o + own8);
#pragma unroll
                for (int ct = 0; ct < 4; ++ct)
                    c.l[s][ct] = *(const double *)(Lc + o + (int64_t)(cb + ct * 16) * 8 + lop8);
            }
        };
        auto mma = [&](const Chunk &c) {
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int ct = 0; ct < 4; ++ct)
                    acc[ct] = __builtin_amdgcn_mfma_f64_16x16x4f64(c.l[s][ct], c.a[s], acc[ct], 0, 0, 0);
        };
        if (cb > 0) {
            const int nc = cb / 8;  // a multiple of eight
            load(0, c0);
            load(1, c1);
            load(2, c2);
            for (int kc = 0;; kc += 4) {
                load(kc + 3, c3);
                mma(c0);
                if (kc + 4 >= nc) break;
                load(kc + 4, c0);
                mma(c1);
                load(kc + 5, c1);
                mma(c2);
                load(kc + 6, c2);
                mma(c3);
            }
            mma(c1);
            mma(c2);
            mma(c3);
        }
#pragma unroll
        for (int ct = 0; ct < 4; ++ct) acc[ct] -= w[ct];
        __syncthreads();  // the diagonal block is in LDS
        if (cb + 64 < b) load_diag(cb + 64);
#pragma unroll 1
        for (int p = 0; p < 4; ++p)
            wave_trsm16(acc, p, Ls, dia[16 * p + gi], inv[16 * p + gi], scratch[wave], gi, gg, [&](int t, double v) {
                const int c = cb + 16 * p + 4 * t;
                *(double *)(X + c * cs + own8) = v;
                if (direct) *(double *)(W + c * cs + own8) = v;
                xmax = fmax(xmax, fabs(v));
                if (!(fabs(v) <= 1.7976931348623157e308)) bad = min(bad, c + gg);
            });
        __syncthreads();  // the diagonal block has been read; the next one reads these columns through other lanes
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) xmax = fmax(xmax, __shfl_xor(xmax, off));
    if (lane == 0) atomicMax(P.pmax + I, (unsigned long long)__double_as_longlong(xmax));
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) bad = min(bad, __shfl_xor(bad, off));
    if (lane == 0 && bad != 0x7FFFFFFF) atomicMin(P.info, (unsigned long long)((int64_t)k * T.b + bad + 1));
}

void launch_trsm_panel(const Tiles &T, const Panel &P, int k, const uint8_t *qmask, hipStream_t st)
{
    const int np = T.nt - k - 1;
    if (np <= 0) return;
    const double *L = (const double *)(T.slots + tile_index(k, k) * T.slot_bytes);
    trsm_kernel<<<dim3(T.b / 64, np), 256, 0, st>>>(T, P, k, L, qmask);
}

// ---------------------------------------------------------------- grouped trailing update
// One launch per class: every work item (I, J) is a b x b tile update
// A_IJ -= L_Ik L_Jk^T from the class's panel copies, or, for a pair of steps,
// A_IJ -= L_Ik L_Jk^T + L_I,k+1 L_J,k+1^T with K = 2b in one accumulation.  Blocks are
// renumbered XCD-aware so the blocks of one item share an L2; an item with
// I == J (SYRK, always FP64) computes its lower blocks only.
// The 128 x 128 FP64 block keeps to 64 registers so that two blocks share a compute
// unit (eight waves per SIMD).
template <typename T, int BM, int BN, int BK, int WM, int WN>
__global__ __launch_bounds__(64 * WM * WN) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 8 && BM == 128 ? 8 : 1)))
void update_cm_kernel(Tiles Tt, const T *panel0, const T *panel1, const int32_t *items)
{
    typedef CMShape<T, BM, BN, BK, WM, WN> S;
    extern __shared__ __align__(16) char smem_raw[];
    const int b = Tt.b;
    const int tmn = b / BM, tnn = b / BN;
    const int64_t lg = xcd_remap(blockIdx.x, gridDim.x);
    const int item = (int)(lg / (tmn * tnn));
    const int rem = (int)(lg % (tmn * tnn));
    const int tm = rem % tmn, tn = rem / tmn;
    const int32_t it = items[item];
    const int I = it >> 16, J = it & 0xFFFF;
    if (I == J && tn * BN > tm * BM + BM - 1) return;
    const int64_t bb = (int64_t)b * b;
    typename CM<T>::acc_t acc[S::MB][S::NB];
#pragma unroll
    for (int m = 0; m < S::MB; ++m)
#pragma unroll
        for (int n = 0; n < S::NB; ++n)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[m][n][v] = 0;
    // small FP64 blocks, bound by latency: what they change is read before the products
    constexpr bool EARLY = sizeof(T) == 8 && BM < 128;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = wave % WM, wn = wave / WM, gi = lane & 15, gg = lane >> 4;
    T *C = (T *)(Tt.slots + tile_index(I, J) * Tt.slot_bytes) + tm * BM + (int64_t)tn * BN * b;
    typename CM<T>::acc_t old[EARLY ? S::MB : 1][EARLY ? S::NB : 1];
    if constexpr (EARLY) {
#pragma unroll
        for (int m = 0; m < S::MB; ++m)
#pragma unroll
            for (int n = 0; n < S::NB; ++n)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    old[m][n][v] = C[wm * (BM / WM) + m * 16 + gi + (wn * (BN / WN) + n * 16 + acc_row<T>(gg, v)) * b];
    }
    // FP64 accumulators hold four rows 4 apart per lane; with the operands
    // swapped each lane owns one row instead, so the stores below cover
    // 16 contiguous doubles per column.  FP32 rows are already contiguous.
    constexpr bool SWAP = sizeof(T) == 8;
    constexpr bool PRIO = sizeof(T) == 4;  // measured: helps FP32, neutral for FP64
    // a pair of steps: K continues over the next panel column; FP64 fetches
    // two K slices ahead (measured +2.3% for the FP64 update alone)
    if constexpr (sizeof(T) == 8)
        cm_block_deep<T, BM, BN, BK, WM, WN, SWAP>(panel0 + I * bb + tm * BM, b, panel0 + J * bb + tn * BN, b, b, acc,
                                                   (T *)smem_raw, panel1 ? panel1 + I * bb + tm * BM : nullptr,
                                                   panel1 ? panel1 + J * bb + tn * BN : nullptr);
    else
        cm_block<T, BM, BN, BK, WM, WN, SWAP, PRIO>(panel0 + I * bb + tm * BM, b, panel0 + J * bb + tn * BN, b, b, acc,
                                                    (T *)smem_raw, panel1 ? panel1 + I * bb + tm * BM : nullptr,
                                                    panel1 ? panel1 + J * bb + tn * BN : nullptr);
#pragma unroll
    for (int m = 0; m < S::MB; ++m)
#pragma unroll
        for (int n = 0; n < S::NB; ++n) {
            if (EARLY) {
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    C[wm * (BM / WM) + m * 16 + gi + (wn * (BN / WN) + n * 16 + acc_row<T>(gg, v)) * b] =
                        old[EARLY ? m : 0][EARLY ? n : 0][v] - acc[m][n][v];
            } else if (SWAP) {
                int r = wm * (BM / WM) + m * 16 + gi, c = wn * (BN / WN) + n * 16;
                T *p = C + r + (int64_t)c * b;
#pragma unroll
                for (int v = 0; v < 4; ++v) p[(int64_t)acc_row<T>(gg, v) * b] -= acc[m][n][v];
            } else {
                int r = wm * (BM / WM) + m * 16, c = wn * (BN / WN) + n * 16 + gi;
                T *p = C + r + (int64_t)c * b;
#pragma unroll
                for (int v = 0; v < 4; ++v) p[acc_row<T>(gg, v)] -= acc[m][n][v];
            }
        }
}

// Up to four panel columns applied in one accumulation (the steps of one or
// two pairs): their copies and scale exponents.
template <typename T> struct PanelSet {
    const T *p[4];
    const int32_t *s[4];  // scale exponents (class q copy of tile I at s[h][I * 4 + q]); unused for the split copies
    const uint8_t *x[4];  // block-scaled FP8: E8M0 block scales of the copies (Panel::p8x)
    int n;
};

template <int KIND, int BM, int BN, int BK, int WM, int WN, bool MX = false>
__global__ __launch_bounds__(64 * WM * WN) void update_rm_kernel(Tiles Tt, PanelSet<typename RM<KIND>::T> ps, int q,
                                                                 const int32_t *items)
{
    typedef RMShape<KIND, BM, BN, BK, WM, WN> S;
    typedef typename RM<KIND>::T T;
    extern __shared__ __align__(16) char smem_raw[];
    const int b = Tt.b;
    const int tmn = b / BM, tnn = b / BN;
    const int64_t lg = xcd_remap(blockIdx.x, gridDim.x);
    const int item = (int)(lg / (tmn * tnn));
    const int rem = (int)(lg % (tmn * tnn));
    const int tm = rem % tmn, tn = rem / tmn;
    const int32_t it = items[item];
    const int I = it >> 16, J = it & 0xFFFF;
    const int64_t bb = (int64_t)b * b;
    float4_t acc[S::MB][S::NB];
#pragma unroll
    for (int m = 0; m < S::MB; ++m)
#pragma unroll
        for (int n = 0; n < S::NB; ++n) acc[m][n] = (float4_t){0.f, 0.f, 0.f, 0.f};
    int tsum = 0;
    if constexpr (MX) {
        // block-scaled copies: the MFMA applies every block's scales, so the
        // steps' products add at their own values
        const int64_t xb = bb / 32, xrow = b / 32;
#pragma nounroll
        for (int h = 0; h < ps.n; ++h)
            rm_block<KIND, BM, BN, BK, WM, WN, true>(ps.p[h] + I * bb + (int64_t)tm * BM * b, b,
                                                     ps.p[h] + J * bb + (int64_t)tn * BN * b, b, b, acc,
                                                     (uint8_t *)smem_raw, ps.x[h] + I * xb + (int64_t)tm * BM * xrow,
                                                     ps.x[h] + J * xb + (int64_t)tn * BN * xrow);
    } else {
        // Scaled copies: the product of step h is acc * 2^-(t_I + t_J) with its own
        // exponent sum.  The steps are taken in decreasing exponent sum (smallest
        // values first); before each later step the accumulator is rescaled down
        // to that step's exponent sum, which is exact and cannot overflow, and
        // the step's product then adds at that scale.
        int ord[4], ts[4];
        for (int h = 0; h < ps.n; ++h) {
            const int t = ps.s[h][I * 4 + q] + ps.s[h][J * 4 + q];
            int pos = h;
            while (pos > 0 && ts[pos - 1] < t) {  // insertion by decreasing t (stable)
                ts[pos] = ts[pos - 1];
                ord[pos] = ord[pos - 1];
                --pos;
            }
            ts[pos] = t;
            ord[pos] = h;
        }
        tsum = ts[0];
#pragma nounroll
        for (int h = 0; h < ps.n; ++h) {
            const T *pn = ps.p[ord[h]];
            if (h) {
                const int t2 = ts[h];
#pragma unroll
                for (int m = 0; m < S::MB; ++m)
#pragma unroll
                    for (int n = 0; n < S::NB; ++n)
#pragma unroll
                        for (int v = 0; v < 4; ++v) acc[m][n][v] = ldexpf(acc[m][n][v], t2 - tsum);
                tsum = t2;
            }
            rm_block<KIND, BM, BN, BK, WM, WN>(pn + I * bb + (int64_t)tm * BM * b, b,
                                               pn + J * bb + (int64_t)tn * BN * b, b, b, acc, (uint8_t *)smem_raw);
        }
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = wave % WM, wn = wave / WM, gi = lane & 15, gg = lane >> 4;
    float *C = (float *)(Tt.slots + tile_index(I, J) * Tt.slot_bytes) + tm * BM + (int64_t)tn * BN * b;
#pragma unroll
    for (int m = 0; m < S::MB; ++m)
#pragma unroll
        for (int n = 0; n < S::NB; ++n) {
            int r = wm * (BM / WM) + m * 16 + 4 * gg, c = wn * (BN / WN) + n * 16 + gi;
            float *p = C + r + (int64_t)c * b;
#pragma unroll
            for (int v = 0; v < 4; ++v) p[v] -= ldexpf(acc[m][n][v], -tsum);
        }
}

// FP32-class update from three-way BF16 splits of the operands (v = hi + mid
// + lo, the FP32 copy exactly): the six significant part products (mid,mid),
// (hi,lo), (lo,hi), (hi,mid), (mid,hi), (hi,hi), smallest first, each over
// the full K on the BF16 MFMA with FP32 accumulation; the three products
// below a float rounding of the result -- (mid,lo), (lo,mid), (lo,lo) -- are
// dropped.  For several steps (a pair, or two pairs) the panels' products of
// one kind follow each other.  Operands: panel + I*3*b*b + part*b*b,
// row-major b x b.
template <int BM, int BN, int BK, int WM, int WN>
__global__ __launch_bounds__(64 * WM * WN) void update_split_kernel(Tiles Tt, PanelSet<uint16_t> ps,
                                                                    const int32_t *items)
{
    typedef RMShape<RM_BF16, BM, BN, BK, WM, WN> S;
    extern __shared__ __align__(16) char smem_raw[];
    const int b = Tt.b;
    const int tmn = b / BM, tnn = b / BN;
    const int64_t lg = xcd_remap(blockIdx.x, gridDim.x);
    const int item = (int)(lg / (tmn * tnn));
    const int rem = (int)(lg % (tmn * tnn));
    const int tm = rem % tmn, tn = rem / tmn;
    const int32_t it = items[item];
    const int I = it >> 16, J = it & 0xFFFF;
    const int64_t bb = (int64_t)b * b, bb3 = 3 * bb;
    float4_t acc[S::MB][S::NB];
#pragma unroll
    for (int m = 0; m < S::MB; ++m)
#pragma unroll
        for (int n = 0; n < S::NB; ++n) acc[m][n] = (float4_t){0.f, 0.f, 0.f, 0.f};
    const int npan = ps.n;
#pragma nounroll
    for (int s = 0; s < 6 * npan; ++s) {
        const int t = s / npan;                      // kind of product, smallest first
        const int pa = (0x010201 >> (4 * t)) & 0xF;  // part of the I operand: 1 0 2 0 1 0
        const int pb = (0x001021 >> (4 * t)) & 0xF;  // part of the J operand: 1 2 0 1 0 0
        const uint16_t *pn = ps.p[s % npan];
        rm_block<RM_BF16, BM, BN, BK, WM, WN>(pn + I * bb3 + pa * bb + (int64_t)tm * BM * b, b,
                                              pn + J * bb3 + pb * bb + (int64_t)tn * BN * b, b, b, acc,
                                              (uint8_t *)smem_raw);
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = wave % WM, wn = wave / WM, gi = lane & 15, gg = lane >> 4;
    float *C = (float *)(Tt.slots + tile_index(I, J) * Tt.slot_bytes) + tm * BM + (int64_t)tn * BN * b;
#pragma unroll
    for (int m = 0; m < S::MB; ++m)
#pragma unroll
        for (int n = 0; n < S::NB; ++n) {
            int r = wm * (BM / WM) + m * 16 + 4 * gg, c = wn * (BN / WN) + n * 16 + gi;
            float *p = C + r + (int64_t)c * b;
#pragma unroll
            for (int v = 0; v < 4; ++v) p[v] -= acc[m][n][v];
        }
}

template <int BM, int BN, int BK, int WM, int WN>
static void launch_split(const Tiles &T_, const PanelSet<uint16_t> &ps, const int32_t *items, int nitems,
                         hipStream_t st)
{
    typedef RMShape<RM_BF16, BM, BN, BK, WM, WN> S;
    auto k = update_split_kernel<BM, BN, BK, WM, WN>;
    static bool attr = false;
    if (!attr) {
        (void)hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)S::SMEM);
        attr = true;
    }
    const int64_t grid = (int64_t)nitems * (T_.b / BM) * (T_.b / BN);
    k<<<(unsigned)grid, S::NTH, S::SMEM, st>>>(T_, ps, items);
}

template <typename T, int BM, int BN, int BK, int WM, int WN>
static void launch_cm(const Tiles &T_, const T *panel0, const T *panel1, const int32_t *items, int nitems,
                      hipStream_t st)
{
    typedef CMShape<T, BM, BN, BK, WM, WN> S;
    auto k = update_cm_kernel<T, BM, BN, BK, WM, WN>;
    static bool attr = false;
    if (!attr) {
        (void)hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)S::SMEM);
        attr = true;
    }
    const int64_t grid = (int64_t)nitems * (T_.b / BM) * (T_.b / BN);
    k<<<(unsigned)grid, S::NTH, S::SMEM, st>>>(T_, panel0, panel1, items);
}

template <int KIND, int BM, int BN, int BK, int WM, int WN, bool MX = false>
static void launch_rm(const Tiles &T_, const PanelSet<typename RM<KIND>::T> &ps, int q, const int32_t *items,
                      int nitems, hipStream_t st)
{
    typedef RMShape<KIND, BM, BN, BK, WM, WN> S;
    constexpr size_t smem = MX ? S::SMEM_MX : S::SMEM;
    auto k = update_rm_kernel<KIND, BM, BN, BK, WM, WN, MX>;
    static bool attr = false;
    if (!attr) {
        (void)hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
        attr = true;
    }
    const int64_t grid = (int64_t)nitems * (T_.b / BM) * (T_.b / BN);
    k<<<(unsigned)grid, S::NTH, smem, st>>>(T_, ps, q, items);
}

// Before a factorization: no bad pivot yet, nothing handed over inside any diagonal tile.
__global__ __launch_bounds__(256) void factor_reset_kernel(unsigned long long *info, int *ctl, int64_t words)
{
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e == 0) *info = ~0ull;
    if (e < words) ctl[e] = 0;
}

void launch_factor_reset(unsigned long long *info, int *ctl, int64_t words, hipStream_t st)
{
    factor_reset_kernel<<<(unsigned)((words + 255) / 256), 256, 0, st>>>(info, ctl, words);
}

// Block shapes per class from a sweep on MI355X (1024 x 1024 tiles):
// FP64 128 x 128 with 16 waves of 32 x 32, FP32 256 x 128 with 8 waves,
// FP16/BF16 256 x 256 with 16 waves, FP8 128 x 128 with 4 waves; tiles of
// 128 fall back to 128 x 128 blocks.
void launch_update(const Tiles &T, const Panel *const *Ps, int npan, int q, const int32_t *items, int nitems,
                   hipStream_t st, bool small)
{
    if (nitems <= 0 || npan < 1 || npan > 4) return;
    // "small": a launch beside the running updates (inside the panel work)
    // uses block shapes whose LDS fits in the slot one finished update block
    // frees; a 1024-thread block with 147 KB of LDS would wait for a whole
    // idle compute unit.
    const bool big = (T.b % 256) == 0 && !small;
    const Panel &P = *Ps[0];
    const Panel *P2 = npan > 1 ? Ps[1] : nullptr;  // the FP64 / FP32-MFMA updates take one pair at most
    switch (q) {
    case P64:
        // a grid of 128 x 128 blocks that does not fill the 512 places on the GPU is
        // bound by one block's chain of loads: blocks of 64 x 64 take a quarter of its
        // products, and stage 32 columns at a time (16 waves; against four waves and 16
        // columns: N = 8,192, tile 1024, 8.35 -> 7.66 ms; N = 4,900, 3.55 -> 3.17).
        // Fewer than 64 blocks would leave compute units idle at 64 x 64 as well: blocks
        // of 32 x 32, 64 columns at a time (N = 1,000, tile 128: 527 -> 457 us)
        if (const int64_t blocks = (int64_t)nitems * (T.b / 128) * (T.b / 128); blocks < 64)
            launch_cm<double, 32, 32, 64, 2, 2>(T, P.p64, P2 ? P2->p64 : nullptr, items, nitems, st);
        else if (blocks < 512)
            launch_cm<double, 64, 64, 32, 4, 4>(T, P.p64, P2 ? P2->p64 : nullptr, items, nitems, st);
        else
            launch_cm<double, 128, 128, 16, 4, 4>(T, P.p64, P2 ? P2->p64 : nullptr, items, nitems, st);
        break;
    case P32:
        if (T.lo32) {
            PanelSet<uint16_t> ps{};
            ps.n = npan;
            for (int h = 0; h < npan; ++h) ps.p[h] = Ps[h]->p32s;
            if (big) launch_split<256, 256, 64, 4, 4>(T, ps, items, nitems, st);
            else launch_split<128, 128, 64, 2, 2>(T, ps, items, nitems, st);
        } else if ((T.b % 256) == 0) {
            launch_cm<float, 256, 128, 16, 4, 2>(T, P.p32, P2 ? P2->p32 : nullptr, items, nitems, st);
        } else {
            launch_cm<float, 128, 128, 16, 2, 2>(T, P.p32, P2 ? P2->p32 : nullptr, items, nitems, st);
        }
        break;
    case P16: {
        PanelSet<uint16_t> ps{};
        ps.n = npan;
        for (int h = 0; h < npan; ++h) {
            ps.p[h] = Ps[h]->p16;
            ps.s[h] = Ps[h]->pscale;
        }
        if (T.lo16 == LO16_BF16) {
            if (big) launch_rm<RM_BF16, 256, 256, 64, 4, 4>(T, ps, q, items, nitems, st);
            else launch_rm<RM_BF16, 128, 128, 64, 2, 2>(T, ps, q, items, nitems, st);
        } else {
            if (big) launch_rm<RM_F16, 256, 256, 64, 4, 4>(T, ps, q, items, nitems, st);
            else launch_rm<RM_F16, 128, 128, 64, 2, 2>(T, ps, q, items, nitems, st);
        }
        break;
    }
    default: {
        PanelSet<uint8_t> ps{};
        ps.n = npan;
        for (int h = 0; h < npan; ++h) {
            ps.p[h] = Ps[h]->p8;
            ps.s[h] = Ps[h]->pscale;
            ps.x[h] = Ps[h]->p8x;
        }
        if (T.lo8) launch_rm<RM_FP8, 128, 128, 128, 2, 2, true>(T, ps, q, items, nitems, st);
        else launch_rm<RM_FP8, 128, 128, 128, 2, 2>(T, ps, q, items, nitems, st);
        break;
    }
    }
}

}  // namespace mpc
