// Solves with Sigma = L L^T on the stored factor: B <- L^-1 B, then
// B <- L^-T B, one launch each.
//
// What bounds it: the factor is read once per direction (N^2 / 2 elements) and
// the N / 64 diagonal blocks form one serial chain.  A launch per diagonal tile
// and a second one for its update of the rest left the whole GPU waiting for
// one wavefront that walked a tile's columns with a global load per column
// (N = 16,384, 16 right-hand sides: 118 ms).  Here a workgroup owns 128 rows
// (forward) or columns (backward) for up to 16 right-hand sides.  It walks the
// 64-wide blocks of the solution in the order in which they become known,
// keeps its sums in registers, then solves its own diagonal block and hands the
// result to the others through B itself.  The factor's elements go from memory
// to registers, each used once, the next block in flight while the current one
// is waited for, so the streaming hides behind the chain or the chain behind it
// (N = 16,384, 16 right-hand sides: 2.17 ms, 8.4 us per 128 rows and direction;
// N = 1,024, one: 4.3 -> 0.1 ms).
//
// Order and progress: a workgroup takes its place in the chain from a ticket
// counter, so it only ever waits for workgroups that started before it: however
// few of them fit on the GPU, the earliest one can always finish.  Solution
// values and the count of finished blocks are written and read with
// device-scope accesses; a workgroup's stores have completed (vmcnt 0, then the
// barrier) before the count is raised.  A wait that lasts longer than
// WAIT_TICKS leaves NaN in the rows it could not solve and ends the launch.
#include "common.h"
#include "launch.h"

namespace mpc {

namespace {

constexpr int NTH = 512, WAVES = 8;      // threads; each wave owns 16 of the 128 rows / columns
constexpr int HB = 64;                   // block of the solution handed on at a time
constexpr int NR = 16;                   // right-hand sides per workgroup
constexpr int LDX = NR + 1, LDD = HB + 1;
constexpr int STEPS = HB / 4;            // K steps of four per block, elements per lane and block
constexpr int NCOPY = 16, STRIDE = 32;   // copies of the finished count, one cache line each
constexpr int CTL = 32 + NCOPY * STRIDE; // words per chunk of right-hand sides and direction
constexpr long long WAIT_TICKS = 3000000000ll;  // 30 s of the 100 MHz counter

struct Ctl {
    unsigned *ticket;  // next place in the chain (shared by the chunks of a launch)
    int *stop;         // set when a wait ran out
    int *done;         // finished blocks: NCOPY copies
};

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

// all of this wave's global stores have completed
__device__ inline void stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

__device__ inline double bcast(double v, int lane)
{
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), lane);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// thread 0: waits until `need` blocks are finished; their number, or -1
__device__ inline int wait_count(const Ctl &c, int copy, int need, bool far)
{
    const int *p = c.done + copy * STRIDE;
    int v = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (v >= need) return v;
    const long long t0 = wall_clock64();
    for (unsigned k = 1;; ++k) {
        if (far) __builtin_amdgcn_s_sleep(16);  // about 1024 cycles: not the next one to run
        v = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (v >= need) return v;
        if ((k & 255) == 0 && (__hip_atomic_load(c.stop, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ||
                               wall_clock64() - t0 > WAIT_TICKS)) {
            __hip_atomic_store(c.stop, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return -1;
        }
    }
}

// A stored tile: base address, class and scale, uniform in the workgroup.
struct TileRef {
    const char *p;
    int cls, t;
};
__device__ inline TileRef tile_ref(const Tiles &T, int I, int J)
{
    return TileRef{T.slots + tile_index(I, J) * T.slot_bytes, I == J ? (int)P64 : (int)T.map[I + (int64_t)J * T.nt],
                   T.tscale[I + (int64_t)J * T.nt]};
}

// STEPS raw codes of a lane, widened only when used so that the loads stay in
// flight.  PAIR (backward): consecutive rows, two codes at off[s].
template <bool PAIR> struct Raw {
    uint64_t u[STEPS];
};
__device__ inline void fetch(const TileRef &R, int off0, int step, Raw<false> &r)
{
    switch (R.cls) {
    case P64:
#pragma unroll
        for (int s = 0; s < STEPS; ++s) r.u[s] = ((const uint64_t *)R.p)[off0 + s * step];
        break;
    case P32:
#pragma unroll
        for (int s = 0; s < STEPS; ++s) r.u[s] = ((const uint32_t *)R.p)[off0 + s * step];
        break;
    case P16:
#pragma unroll
        for (int s = 0; s < STEPS; ++s) r.u[s] = ((const uint16_t *)R.p)[off0 + s * step];
        break;
    default:
#pragma unroll
        for (int s = 0; s < STEPS; ++s) r.u[s] = ((const uint8_t *)R.p)[off0 + s * step];
        break;
    }
}
typedef uint64_t u64x2 __attribute__((ext_vector_type(2)));
// pairs of rows 8 apart: off0 is even and tiles are 16-byte aligned
__device__ inline void fetch(const TileRef &R, int off0, Raw<true> &r)
{
    switch (R.cls) {
    case P64:
#pragma unroll
        for (int s = 0; s < STEPS / 2; ++s) {
            const u64x2 v = *(const u64x2 *)((const uint64_t *)R.p + off0 + 8 * s);
            r.u[2 * s] = v[0];
            r.u[2 * s + 1] = v[1];
        }
        break;
    case P32:
#pragma unroll
        for (int s = 0; s < STEPS / 2; ++s) {
            const uint64_t v = *(const uint64_t *)((const uint32_t *)R.p + off0 + 8 * s);
            r.u[2 * s] = v & 0xFFFFFFFFu;
            r.u[2 * s + 1] = v >> 32;
        }
        break;
    case P16:
#pragma unroll
        for (int s = 0; s < STEPS / 2; ++s) {
            const uint32_t v = *(const uint32_t *)((const uint16_t *)R.p + off0 + 8 * s);
            r.u[2 * s] = v & 0xFFFFu;
            r.u[2 * s + 1] = v >> 16;
        }
        break;
    default:
#pragma unroll
        for (int s = 0; s < STEPS / 2; ++s) {
            const uint16_t v = *(const uint16_t *)((const uint8_t *)R.p + off0 + 8 * s);
            r.u[2 * s] = v & 0xFFu;
            r.u[2 * s + 1] = v >> 8;
        }
        break;
    }
}
__device__ inline double widen(uint64_t u, const TileRef &R, int lo16)
{
    return R.cls == P64 ? __longlong_as_double((long long)u) : decode_class((uint32_t)u, R.cls, lo16, R.t);
}

// The sums of a lane.  ONE (a single right-hand side): row gi of the wave's 16,
// the terms of K group gg; else MFMA accumulators, rows gg + 4v, right-hand side gi.
template <bool ONE> struct Sum {
    double4_t v;
    __device__ inline void zero() { v = (double4_t){0.0, 0.0, 0.0, 0.0}; }
    __device__ inline void add(double a, const double *x, int k, int gi)
    {
        if (ONE) v[0] += a * x[k];
        else v = __builtin_amdgcn_mfma_f64_16x16x4f64(a, x[k * LDX + gi], v, 0, 0, 0);
    }
};

}  // namespace

// Finished counts, tickets and stop words of both directions to zero (a
// kernel, so that a captured solve replays).
__global__ __launch_bounds__(256) void solve_reset_kernel(int *ctl, int words)
{
    for (int i = blockIdx.x * 256 + threadIdx.x; i < words; i += gridDim.x * 256) ctl[i] = 0;
}

// FWD: rows row0 .. row0 + 127 of L y = b, blocks in increasing order; else
// columns of L^T x = y, blocks in decreasing order.  Diagonal blocks are solved
// as D^-1 (L D^-1)^-1 (forward) or (D^-1 L^T)^-1 D^-1 (backward), D the
// diagonal of the block: scaling the columns (rows) beforehand leaves one
// broadcast and one fused multiply-add per step on the chain, the divisions
// outside it.
template <bool FWD, bool ONE>
__global__ __launch_bounds__(NTH) void solve_kernel(Tiles T, double *B, int64_t ldb, int nrhs, int *ctl)
{
    __shared__ double xs[2][HB * LDX];
    __shared__ double xh[HB * LDX];        // this workgroup's first solved half
    __shared__ double ds[2][HB * LDD];     // scaled diagonal blocks, ds[h][c * LDD + lane]
    __shared__ double rs[NR][HB + 1];      // right-hand side of the half being solved
    __shared__ double dg[2 * HB];
    __shared__ int s_word;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, gi = lane & 15, gg = lane >> 4;
    const int b = T.b, nchunk = (nrhs + NR - 1) / NR, nblk = (int)((T.n + 127) / 128);
    if (tid == 0) s_word = (int)atomicAdd((unsigned *)ctl, 1u);
    __syncthreads();
    const int place = s_word;
    __syncthreads();
    const int chunk = place % nchunk, seq = place / nchunk;
    const int blk = FWD ? seq : nblk - 1 - seq;
    const Ctl c{(unsigned *)ctl, ctl + 1, ctl + 32 + chunk * (NCOPY * STRIDE)};
    const int copy = seq % NCOPY;
    const int j0 = chunk * NR, nr = min(NR, nrhs - j0);
    const int64_t row0 = (int64_t)blk * 128;
    const int I = (int)(row0 / b), lr = (int)(row0 - (int64_t)I * b);
    double *Bc = B + (int64_t)j0 * ldb;

    // own right-hand side, diagonal blocks and the block between them, all read ahead of the chain
    double rb[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int r = ONE ? gi : gg + 4 * v, q = ONE ? 0 : gi;
        const int64_t i = row0 + wave * 16 + r;
        rb[v] = (i < T.n && q < nr && (!ONE || v == 0)) ? Bc[i + (int64_t)q * ldb] : 0.0;
    }
    const TileRef D = tile_ref(T, I, I);
    const double *Dd = (const double *)D.p + lr + (int64_t)lr * b;
    if (tid < 2 * HB) dg[tid] = Dd[tid + (int64_t)tid * b];
    __syncthreads();
    for (int e = tid; e < 2 * HB * HB; e += NTH) {
        const int h = e / (HB * HB), r = e % HB, q = (e / HB) % HB;
        const double l = Dd[h * HB + r + (int64_t)(h * HB + q) * b];
        if (FWD) ds[h][q * LDD + r] = r > q ? l / dg[h * HB + q] : 0.0;
        else ds[h][r * LDD + q] = q < r ? l / dg[h * HB + q] : 0.0;
    }
    // the waves of the second half to be solved (rows 64.. forward, columns 0..63 backward)
    const bool second = FWD ? wave >= WAVES / 2 : wave < WAVES / 2;
    Raw<!FWD> mid;
    if constexpr (FWD) {
        if (second) fetch(D, lr + wave * 16 + gi + (lr + gg) * b, 4 * b, mid);
    } else {
        if (second) fetch(D, lr + HB + 2 * gg + (lr + wave * 16 + gi) * b, mid);
    }

    Sum<ONE> acc;
    acc.zero();
    const int first = FWD ? 0 : 2 * nblk - 1, count = 2 * seq;  // blocks before this workgroup's own
    auto ref = [&](int k) {  // the tile holding step k's block
        const int64_t q0 = (int64_t)(FWD ? k : first - k) * HB;
        const int K = (int)(q0 / b);
        return FWD ? tile_ref(T, I, K) : tile_ref(T, K, I);
    };
    auto fetch_step = [&](int k, const TileRef &R, Raw<!FWD> &r) {
        const int64_t q0 = (int64_t)(FWD ? k : first - k) * HB;
        const int lq = (int)(q0 % b);
        if constexpr (FWD) fetch(R, lr + wave * 16 + gi + (lq + gg) * b, 4 * b, r);
        else fetch(R, lq + 2 * gg + (lr + wave * 16 + gi) * b, r);
    };
    auto product = [&](const Raw<!FWD> &r, const TileRef &R, const double *x) {
#pragma unroll
        for (int s = 0; s < STEPS; ++s) {
            const int k = FWD ? 4 * s + gg : 8 * (s >> 1) + 2 * gg + (s & 1);
            acc.add(widen(r.u[s], R, T.lo16), x, k, gi);
        }
    };
    int seen = 0;
    Raw<!FWD> ra, rn;
    TileRef Ra = D, Rn = D;
    if (count > 0) {
        Ra = ref(0);
        fetch_step(0, Ra, ra);
    }
    for (int k = 0; k < count; ++k) {
        if (k + 1 < count) {
            Rn = ref(k + 1);
            fetch_step(k + 1, Rn, rn);
        }
        if (k >= seen) {
            if (tid == 0) s_word = wait_count(c, copy, k + 1, count - k > 4);
            __syncthreads();
            seen = s_word;
            if (seen < 0) {
                for (int e = tid; e < 128 * nr; e += NTH) {
                    const int64_t i = row0 + e % 128;
                    if (i < T.n) st_dev(Bc + i + (int64_t)(e / 128) * ldb, __builtin_nan(""));
                }
                return;
            }
        }
        double *x = xs[k & 1];
        const int64_t q0 = (int64_t)(FWD ? k : first - k) * HB;
        for (int e = tid; e < (ONE ? HB : HB * NR); e += NTH) {
            const int r = e % HB, q = e / HB;
            const double v = (q < nr && q0 + r < T.n) ? ld_dev(Bc + q0 + r + (int64_t)q * ldb) : 0.0;
            x[ONE ? r : r * LDX + q] = v;
        }
        __syncthreads();
        product(ra, Ra, x);
        ra = rn;
        Ra = Rn;
    }

    // the two halves of the own block
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        const int h = FWD ? half : 1 - half;
        const bool mine = half == 0 ? !second : second;
        if (half == 1 && second) product(mid, D, xh);
        if (mine) {
            const int w = wave - (FWD ? half : 1 - half) * (WAVES / 2);
            if (ONE) {
                double s = acc.v[0];
                s += __shfl_xor(s, 16);
                s += __shfl_xor(s, 32);
                if (gg == 0) rs[0][w * 16 + gi] = rb[0] - s;
            } else {
#pragma unroll
                for (int v = 0; v < 4; ++v) rs[gi][w * 16 + gg + 4 * v] = rb[v] - acc.v[v];
            }
        }
        __syncthreads();
        if (!ONE || wave == 0) {
            constexpr int NQ = ONE ? 1 : NR / WAVES;
            double v[NQ];
            const double d = dg[h * HB + lane];
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                v[q] = rs[wave * NQ + q][lane];
                if (!FWD) v[q] = v[q] / d;
            }
            const double *dl = ds[h] + lane;
#pragma unroll
            for (int t = 0; t < HB - 1; ++t) {
                const int cc = FWD ? t : HB - 1 - t;
                const double l = dl[cc * LDD];
#pragma unroll
                for (int q = 0; q < NQ; ++q) v[q] -= l * bcast(v[q], cc);
            }
            const int64_t i = row0 + h * HB + lane;
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                const int rq = wave * NQ + q;
                if (FWD) v[q] = v[q] / d;
                if (i < T.n && rq < nr) st_dev(Bc + i + (int64_t)rq * ldb, v[q]);
                xh[ONE ? lane : lane * LDX + rq] = v[q];
            }
            stores_done();
        }
        __syncthreads();
        if (tid < NCOPY)
            __hip_atomic_store(c.done + tid * STRIDE, count + half + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// Right-hand sides per launch: 16 chunks share a launch, each with its own chain.
constexpr int MAXCHUNK = 16;

size_t solve_ctl_bytes() { return (size_t)2 * (32 + MAXCHUNK * NCOPY * STRIDE) * sizeof(int); }

void launch_solve(const Tiles &T, double *B, int64_t ldb, int nrhs, int *ctl, hipStream_t st)
{
    const int words = (int)(solve_ctl_bytes() / sizeof(int));
    const unsigned nblk = (unsigned)((T.n + 127) / 128);
    for (int j0 = 0; j0 < nrhs; j0 += MAXCHUNK * NR) {
        const int nr = nrhs - j0 < MAXCHUNK * NR ? nrhs - j0 : MAXCHUNK * NR;
        double *Bj = B + (int64_t)j0 * ldb;
        const unsigned grid = nblk * (unsigned)((nr + NR - 1) / NR);
        int *bwd = ctl + words / 2;
        solve_reset_kernel<<<16, 256, 0, st>>>(ctl, words);
        if (nr == 1) {
            solve_kernel<true, true><<<grid, NTH, 0, st>>>(T, Bj, ldb, nr, ctl);
            solve_kernel<false, true><<<grid, NTH, 0, st>>>(T, Bj, ldb, nr, bwd);
        } else {
            solve_kernel<true, false><<<grid, NTH, 0, st>>>(T, Bj, ldb, nr, ctl);
            solve_kernel<false, false><<<grid, NTH, 0, st>>>(T, Bj, ldb, nr, bwd);
        }
    }
}

}  // namespace mpc
