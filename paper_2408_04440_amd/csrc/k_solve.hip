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
// result to the others through a mailbox.  The factor's elements go from memory
// to registers, each used once, the next block in flight while the current one
// is waited for, so the streaming hides behind the chain or the chain behind it
// (N = 16,384: 16 right-hand sides 2.16 -> 1.80 ms, 7.0 us per 128 rows and
// direction, where counts handed the blocks on and eight waves broadcast each
// solved value; mixed classes 2.42 -> 1.78; one right-hand side 1.50 -> 1.36).
//
// Order and progress: a workgroup takes its place in the chain from a ticket
// counter, so it only ever waits for workgroups that started before it: however
// few of them fit on the GPU, the earliest one can always finish.  The mailbox
// has a place for every value of the solution, marked EMPTY before the launch,
// and is written and read with device-scope accesses.  The workgroups next in the
// chain poll the values themselves (a count raised once they are visible, polled,
// and the values read after it are three trips to memory instead of one); the
// others, further back, wait for a count of finished blocks, raised when a
// workgroup's stores have completed (vmcnt 0, then the barrier), and poll it at
// leisure.  Workgroups that follow on the values alone can be done before the one
// they got them from has raised the count, so it only ever goes up.  A wait that lasts longer than its limit leaves NaN in the rows it
// could not solve, ends the launch and sets the caller's word.
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
constexpr int NEAR = 4;                  // blocks before its own that a workgroup polls for themselves
constexpr unsigned long long EMPTY = 0x7FF85EED0BADF00Dull;  // a NaN that no stored solution value has

struct Ctl {
    unsigned *ticket;  // next place in the chain (shared by the chunks of a launch)
    int *stop;         // set when a wait ran out
    int *done;         // finished blocks: NCOPY copies
    int *late;         // host memory: the same, for the caller
    long long wait;    // the limit, in ticks
};

__device__ inline unsigned long long ld_mail(const unsigned long long *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline void st_mail(unsigned long long *p, double v)
{
    unsigned long long u = (unsigned long long)__double_as_longlong(v);
    if (u == EMPTY) u ^= 1;  // stays a NaN
    __hip_atomic_store(p, u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One column of the triangle: v[t][p] -= (lane JJ of the row of 16's v[S][p]) * l[t]
// for the 16-row tiles t behind S in the order of the solve, then for S itself: DPP
// multiply-adds, 5 cycles each (as broadcasts and multiply-adds of their own a
// step costs the vector unit three times that).  The s_nop covers the wait states
// between the last writes of v[S] and their DPP reads, which the compiler does
// not see here.
#define MPC_FM(d, s, l) "\n\tv_fmac_f64_dpp %[" d "], -%[" s "], %[" l "] row_newbcast:%[jj] row_mask:0xf bank_mask:0xf"
template <int JJ, int NB> __device__ inline void column(double (&x)[1], double *const (&y)[3], const double (&l)[4])
{
    if constexpr (NB == 0)
        asm("s_nop 1" MPC_FM("x", "x", "k") : [x] "+v"(x[0]) : [k] "v"(l[0]), [jj] "n"(JJ));
    else if constexpr (NB == 1)
        asm("s_nop 1" MPC_FM("a", "x", "ka") MPC_FM("x", "x", "k")
            : [x] "+v"(x[0]), [a] "+v"(y[0][0])
            : [k] "v"(l[0]), [ka] "v"(l[1]), [jj] "n"(JJ));
    else if constexpr (NB == 2)
        asm("s_nop 1" MPC_FM("a", "x", "ka") MPC_FM("b", "x", "kb") MPC_FM("x", "x", "k")
            : [x] "+v"(x[0]), [a] "+v"(y[0][0]), [b] "+v"(y[1][0])
            : [k] "v"(l[0]), [ka] "v"(l[1]), [kb] "v"(l[2]), [jj] "n"(JJ));
    else
        asm("s_nop 1" MPC_FM("a", "x", "ka") MPC_FM("b", "x", "kb") MPC_FM("c", "x", "kc") MPC_FM("x", "x", "k")
            : [x] "+v"(x[0]), [a] "+v"(y[0][0]), [b] "+v"(y[1][0]), [c] "+v"(y[2][0])
            : [k] "v"(l[0]), [ka] "v"(l[1]), [kb] "v"(l[2]), [kc] "v"(l[3]), [jj] "n"(JJ));
}
template <int JJ, int NB> __device__ inline void column(double (&x)[2], double *const (&y)[3], const double (&l)[4])
{
    if constexpr (NB == 0)
        asm("s_nop 1" MPC_FM("x", "x", "k") MPC_FM("z", "z", "k")
            : [x] "+v"(x[0]), [z] "+v"(x[1])
            : [k] "v"(l[0]), [jj] "n"(JJ));
    else if constexpr (NB == 1)
        asm("s_nop 1" MPC_FM("a", "x", "ka") MPC_FM("d", "z", "ka") MPC_FM("x", "x", "k") MPC_FM("z", "z", "k")
            : [x] "+v"(x[0]), [z] "+v"(x[1]), [a] "+v"(y[0][0]), [d] "+v"(y[0][1])
            : [k] "v"(l[0]), [ka] "v"(l[1]), [jj] "n"(JJ));
    else if constexpr (NB == 2)
        asm("s_nop 1" MPC_FM("a", "x", "ka") MPC_FM("d", "z", "ka") MPC_FM("b", "x", "kb") MPC_FM("e", "z", "kb")
            MPC_FM("x", "x", "k") MPC_FM("z", "z", "k")
            : [x] "+v"(x[0]), [z] "+v"(x[1]), [a] "+v"(y[0][0]), [d] "+v"(y[0][1]), [b] "+v"(y[1][0]), [e] "+v"(y[1][1])
            : [k] "v"(l[0]), [ka] "v"(l[1]), [kb] "v"(l[2]), [jj] "n"(JJ));
    else
        asm("s_nop 1" MPC_FM("a", "x", "ka") MPC_FM("d", "z", "ka") MPC_FM("b", "x", "kb") MPC_FM("e", "z", "kb")
            MPC_FM("c", "x", "kc") MPC_FM("f", "z", "kc") MPC_FM("x", "x", "k") MPC_FM("z", "z", "k")
            : [x] "+v"(x[0]), [z] "+v"(x[1]), [a] "+v"(y[0][0]), [d] "+v"(y[0][1]), [b] "+v"(y[1][0]), [e] "+v"(y[1][1]),
              [c] "+v"(y[2][0]), [f] "+v"(y[2][1])
            : [k] "v"(l[0]), [ka] "v"(l[1]), [kb] "v"(l[2]), [kc] "v"(l[3]), [jj] "n"(JJ));
}
#undef MPC_FM

// One wave solves a 64 x 64 unit triangle for P right-hand sides per row of 16
// lanes: v[t][p], rows 16 t + gi; dl: column c at dl[c * LDD + row], zero on and
// beyond the diagonal.  Columns in groups of 12 to 16 entries a lane, the next
// group's on their way from LDS meanwhile.
constexpr int NG = 11;
__device__ constexpr int group_at(int g) { return g < 8 ? 4 * g : g < 10 ? 32 + 8 * (g - 8) : 48 + 16 * (g - 10); }

template <bool FWD, int P> __device__ inline void solve64(double (&v)[4][P], const double *dl, int gi)
{
    double l[2][16][4];  // [set][column][own tile, then those behind it]
    auto load = [&](auto ig) {
        constexpr int g = decltype(ig)::value;
        static_for<0, group_at(g + 1) - group_at(g)>([&](auto ic) {
            constexpr int k = decltype(ic)::value, at = group_at(g) + k, c = FWD ? at : HB - 1 - at, S = c / 16;
            constexpr int NB = FWD ? 3 - S : S;
#pragma unroll
            for (int t = 0; t <= NB; ++t) l[g & 1][k][t] = dl[c * LDD + 16 * (FWD ? S + t : S - t) + gi];
        });
    };
    load(std::integral_constant<int, 0>{});
    static_for<0, NG>([&](auto ig) {
        constexpr int g = decltype(ig)::value;
        if constexpr (g + 1 < NG) load(std::integral_constant<int, g + 1>{});
        __builtin_amdgcn_sched_barrier(0);
        static_for<0, group_at(g + 1) - group_at(g)>([&](auto ic) {
            constexpr int k = decltype(ic)::value, at = group_at(g) + k, c = FWD ? at : HB - 1 - at, S = c / 16;
            constexpr int NB = FWD ? 3 - S : S, D = FWD ? 1 : -1;
            double *const y[3] = {v[NB > 0 ? S + D : S], v[NB > 1 ? S + 2 * D : S], v[NB > 2 ? S + 3 * D : S]};
            column<c % 16, NB>(v[S], y, l[g & 1][k]);
        });
        __builtin_amdgcn_sched_barrier(0);
    });
}

// Quotients by reciprocals (div_by) where nothing in them can leave the range of
// normal numbers: dividend and divisor both in_range.
__device__ inline bool in_range(double v)
{
    const unsigned e = ((unsigned)((unsigned long long)__double_as_longlong(v) >> 52)) & 0x7FFu;
    return e - 523u < 1000u;  // 2^-500 <= |v| < 2^500
}
// a wait has run out, here or elsewhere in this direction
__device__ inline bool out_of_time(const Ctl &c, long long t0)
{
    if (!__hip_atomic_load(c.stop, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) && wall_clock64() - t0 <= c.wait)
        return false;
    __hip_atomic_store(c.stop, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(c.late, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    return true;
}

// Raises a count of finished blocks to v, whatever a later workgroup has made of it.
__host__ __device__ inline void raise_count(int *p, int v)
{
    __hip_atomic_fetch_max(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// thread 0: waits until `need` blocks are finished; their number, or -1
__device__ inline int wait_count(const Ctl &c, int copy, int need)
{
    const int *p = c.done + copy * STRIDE;
    int v = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (v >= need) return v;
    const long long t0 = wall_clock64();
    for (unsigned k = 1;; ++k) {
        __builtin_amdgcn_s_sleep(16);  // about 1024 cycles: not the next one to run
        v = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (v >= need) return v;
        if ((k & 255) == 0 && out_of_time(c, t0)) return -1;
    }
}

// one value of the mailbox, waited for; false if it did not come
__device__ inline bool receive(const Ctl &c, const unsigned long long *p, unsigned long long &u)
{
    if (u != EMPTY) return true;
    const long long t0 = wall_clock64();
    for (unsigned k = 1;; ++k) {
        u = ld_mail(p);
        if (u != EMPTY) return true;
        if ((k & 255) == 0 && out_of_time(c, t0)) return false;
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
// flight.  PAIR (backward): consecutive rows, two to a load.
template <bool PAIR> struct Raw {
    uint64_t u[STEPS];
};
// single rows: the aligned 8 bytes that hold each, by the same load for every class
__device__ inline void fetch(const TileRef &R, int off0, int step, Raw<false> &r)
{
    const int sh = class_shift(R.cls);
#pragma unroll
    for (int s = 0; s < STEPS; ++s) r.u[s] = *(const uint64_t *)(R.p + (((off0 + s * step) << sh) & ~7));
}
// pairs of rows 8 apart (off0 even), by the same 16-byte load for every class
__device__ inline void fetch(const TileRef &R, int off0, Raw<true> &r)
{
    const int sh = class_shift(R.cls);
#pragma unroll
    for (int s = 0; s < STEPS / 2; ++s) {
        const ulonglong2 v = load_pair16(R.p, (off0 + 8 * s) << sh);
        r.u[2 * s] = v.x;
        r.u[2 * s + 1] = v.y;
    }
}

// The STEPS values of a lane; a loop per class, so that no branch stands between
// the products.  gi (single rows) or gg (pairs) places the codes in the bytes read
// with them: columns, blocks and a wave's rows start at multiples of 16 values.
template <int CLS, bool PAIR>
__device__ inline void widen(const Raw<PAIR> &r, int gi, int gg, int lo16, int t, double (&a)[STEPS])
{
#pragma unroll
    for (int s = 0; s < STEPS; ++s) {
        if (CLS == P64) {
            a[s] = __longlong_as_double((long long)r.u[s]);
        } else {
            constexpr int SH = CLS == P32 ? 2 : CLS == P16 ? 1 : 0, BITS = 8 << SH;
            uint32_t c;
            if (PAIR) {
                const uint64_t u = pair_codes(make_ulonglong2(r.u[s & ~1], r.u[s | 1]), (2 * gg + 4 * (s & ~1)) << SH);
                c = (uint32_t)(u >> (BITS * (s & 1)));
            } else {
                c = (uint32_t)(r.u[s] >> (8 * ((gi << SH) & 7)));
            }
            a[s] = decode_class(BITS == 32 ? c : c & ((1u << (BITS & 31)) - 1), CLS, lo16, t);
        }
    }
}

// a and b with b's first and a's second 32 lanes exchanged, or b's even and a's odd rows of 16.
template <int LANES> __device__ inline void swap_lanes(double &a, double &b)
{
    const unsigned long long u = (unsigned long long)__double_as_longlong(a), v = (unsigned long long)__double_as_longlong(b);
    const auto lo = LANES == 32 ? __builtin_amdgcn_permlane32_swap((unsigned)u, (unsigned)v, false, false)
                                : __builtin_amdgcn_permlane16_swap((unsigned)u, (unsigned)v, false, false);
    const auto hi = LANES == 32 ? __builtin_amdgcn_permlane32_swap((unsigned)(u >> 32), (unsigned)(v >> 32), false, false)
                                : __builtin_amdgcn_permlane16_swap((unsigned)(u >> 32), (unsigned)(v >> 32), false, false);
    a = __longlong_as_double((long long)((unsigned long long)hi[0] << 32 | lo[0]));
    b = __longlong_as_double((long long)((unsigned long long)hi[1] << 32 | lo[1]));
}
template <int LANES> __device__ inline double swap_add(double a, double b)
{
    swap_lanes<LANES>(a, b);
    return a + b;
}
// over the four rows of 16 lanes
__device__ inline double sum_rows(double v)
{
    v = swap_add<32>(v, v);
    return swap_add<16>(v, v);
}

// The running value of a lane: products less right-hand side.  ONE (a single
// right-hand side): row gi of the wave's 16, the same in every row of lanes; else MFMA
// accumulators, rows gg + 4v, right-hand side gi.  The products of a block of 64 are
// summed from zero, in runs of neighbours, and added once: the terms of such a sum
// nearly cancel from one to the next (a solve undoes what the correlation of
// neighbours did), and sums over every other term, or every other four, lose what
// cancels (N = 1,444, correlation length 20: 9 times the error, and 1% of the time
// saved, 3% with one right-hand side).
template <bool FWD, bool ONE> struct Sum {
    double4_t t;
    // column (row) of the block that a[s] belongs to
    static __device__ inline int place(int s, int gg)
    {
        if (ONE) return FWD ? 16 * gg + s : 8 * (s >> 1) + 2 * gg + (s & 1);
        return FWD ? 4 * s + gg : 8 * (s >> 1) + 4 * (s & 1) + 2 * (gg & 1) + (gg >> 1);
    }
    // a: the lane's elements as they were read
    __device__ inline void add(double (&a)[STEPS], const double (&x)[STEPS])
    {
        if constexpr (!ONE) {
            double4_t v = {0.0, 0.0, 0.0, 0.0}, w = v;  // the halves of the block, in turn: always a product to issue
            if constexpr (!FWD) {  // pairs of rows: four neighbours to a product
#pragma unroll
                for (int s = 0; s < STEPS; s += 2) swap_lanes<32>(a[s], a[s + 1]);
            }
#pragma unroll
            for (int s = 0; s < STEPS / 2; ++s) {
                v = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s], x[s], v, 0, 0, 0);
                w = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s + STEPS / 2], x[s + STEPS / 2], w, 0, 0, 0);
            }
            t += v + w;
        } else if constexpr (FWD) {
            double v = 0.0, w = 0.0;
#pragma unroll
            for (int s = 0; s < STEPS / 2; ++s) {
                v += a[s] * x[s];
                w += a[s + STEPS / 2] * x[s + STEPS / 2];
            }
            t[0] += sum_rows(v + w);
        } else {
            double p[STEPS / 2];  // pairs; then runs of eight rows, a different one in each row of lanes
#pragma unroll
            for (int j = 0; j < STEPS / 2; ++j) p[j] = a[2 * j] * x[2 * j] + a[2 * j + 1] * x[2 * j + 1];
            const double q0 = swap_add<16>(swap_add<32>(p[0], p[1]), swap_add<32>(p[2], p[3]));
            const double q1 = swap_add<16>(swap_add<32>(p[4], p[5]), swap_add<32>(p[6], p[7]));
            t[0] += sum_rows(q0 + q1);
        }
    }
};

}  // namespace

// Finished counts, tickets and stop words of both directions to zero, their
// mailboxes to EMPTY (a kernel, so that a captured solve replays).
__global__ __launch_bounds__(256) void solve_reset_kernel(int *ctl, int words, unsigned long long *mail, int64_t places)
{
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x, nt = (int64_t)gridDim.x * 256;
    for (int64_t i = t; i < words; i += nt) ctl[i] = 0;
    for (int64_t i = t; i < places; i += nt) mail[i] = EMPTY;
}

// FWD: rows row0 .. row0 + 127 of L y = b, blocks in increasing order; else
// columns of L^T x = y, blocks in decreasing order.  Diagonal blocks are solved
// as D^-1 (L D^-1)^-1 (forward) or (D^-1 L^T)^-1 D^-1 (backward), D the
// diagonal of the block: scaling the columns (rows) beforehand leaves one
// broadcast and one fused multiply-add per step on the chain, the divisions
// outside it.
template <bool FWD, bool ONE>
__global__ __launch_bounds__(NTH) void solve_kernel(Tiles T, double *B, int64_t ldb, int nrhs, int *ctl,
                                                     unsigned long long *mail, int *late, long long wait)
{
    __shared__ double xs[2][HB * LDX];
    __shared__ double xh[HB * LDX];        // this workgroup's first solved half
    __shared__ double ds[2][HB * LDD];     // scaled diagonal blocks, ds[h][c * LDD + lane]
    __shared__ double rs[NR][HB + 1];      // right-hand side of the half being solved
    __shared__ double dg[2 * HB], rg[2 * HB];  // diagonal and its reciprocal
    __shared__ int s_word, s_late;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, gi = lane & 15, gg = lane >> 4;
    const int b = T.b, nchunk = (nrhs + NR - 1) / NR, nblk = (int)((T.n + 127) / 128);
    if (tid == 0) {
        s_word = (int)atomicAdd((unsigned *)ctl, 1u);
        s_late = 0;
    }
    __syncthreads();
    const int place = s_word;
    __syncthreads();
    const int chunk = place % nchunk, seq = place / nchunk;
    const int blk = FWD ? seq : nblk - 1 - seq;
    const Ctl c{(unsigned *)ctl, ctl + 1, ctl + 32 + chunk * (NCOPY * STRIDE), late, wait};
    const int copy = seq % NCOPY;
    const int j0 = chunk * NR, nr = min(NR, nrhs - j0);
    const int64_t row0 = (int64_t)blk * 128;
    const int I = (int)(row0 / b), lr = (int)(row0 - (int64_t)I * b);
    double *Bc = B + (int64_t)j0 * ldb;
    constexpr int PER = HB * (ONE ? 1 : NR);  // places of a 64-block: right-hand side by right-hand side
    unsigned long long *mc = mail + (int64_t)chunk * 2 * nblk * PER;

    // own right-hand side, diagonal blocks and the block between them, all read ahead of the chain
    Sum<FWD, ONE> acc;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int r = ONE ? gi : gg + 4 * v, q = ONE ? 0 : gi;
        const int64_t i = row0 + wave * 16 + r;
        acc.t[v] = (i < T.n && q < nr && (!ONE || v == 0)) ? -Bc[i + (int64_t)q * ldb] : 0.0;
    }
    const TileRef D = tile_ref(T, I, I);
    const double *Dd = (const double *)D.p + lr + (int64_t)lr * b;
    bool plain = true;
    if (tid < 2 * HB) {
        const double d = Dd[tid + (int64_t)tid * b];
        dg[tid] = d;
        rg[tid] = 1.0 / d;
        plain = in_range(d);
    }
    plain = __syncthreads_and(plain);
    for (int e = tid; e < 2 * HB * HB; e += NTH) {
        const int h = e / (HB * HB), r = e % HB, q = (e / HB) % HB;
        const double l = Dd[h * HB + r + (int64_t)(h * HB + q) * b];
        if (FWD) ds[h][q * LDD + r] = r > q ? l / dg[h * HB + q] : 0.0;
        else ds[h][r * LDD + q] = q < r ? l / dg[h * HB + q] : 0.0;
    }
    // the waves of the second half to be solved (rows 64.. forward, columns 0..63 backward)
    const bool second = FWD ? wave >= WAVES / 2 : wave < WAVES / 2;
    // the rows solved first go first: what they wait for is on the chain
    if (!second) __builtin_amdgcn_s_setprio(2);
    const int first = FWD ? 0 : 2 * nblk - 1, count = 2 * seq;  // blocks before this workgroup's own
    // the tile holding step k's block; its class is read once per tile, as a read of
    // it waits for the pieces sent for before
    int at = -1;
    TileRef Rt = D;
    auto ref = [&](int k) {
        const int K = (int)((int64_t)(FWD ? k : first - k) * HB / b);
        if (K != at) {
            at = K;
            Rt = FWD ? tile_ref(T, I, K) : tile_ref(T, K, I);
            Rt.cls = __builtin_amdgcn_readfirstlane(Rt.cls);
        }
        return Rt;
    };
    auto fetch_step = [&](int k, const TileRef &R, Raw<!FWD> &r) {
        const int64_t q0 = (int64_t)(FWD ? k : first - k) * HB;
        const int lq = (int)(q0 % b);
        if constexpr (FWD) fetch(R, lr + wave * 16 + gi + (lq + (ONE ? 16 : 1) * gg) * b, (ONE ? 1 : 4) * b, r);
        else fetch(R, lq + 2 * gg + (lr + wave * 16 + gi) * b, r);
    };
    auto product = [&](const Raw<!FWD> &r, const TileRef &R, const double *x) {
        // all of the operands first: neither a branch on the class nor a wait between the products
        double a[STEPS], xk[STEPS];
#pragma unroll
        for (int s = 0; s < STEPS; ++s) {
            const int k = Sum<FWD, ONE>::place(s, gg);
            xk[s] = x[ONE ? k : k * LDX + gi];
        }
        // FP64 by itself: joined with the other classes its values are moved, and the
        // move waits for the pieces sent for meanwhile as well
        if (R.cls == P64) {
            widen<P64>(r, gi, gg, T.lo16, R.t, a);
            acc.add(a, xk);
            return;
        }
        switch (R.cls) {
        case P32: widen<P32>(r, gi, gg, T.lo16, R.t, a); break;
        case P16: widen<P16>(r, gi, gg, T.lo16, R.t, a); break;
        default: widen<P8>(r, gi, gg, T.lo16, R.t, a); break;
        }
        acc.add(a, xk);
    };
    auto give_up = [&]() {
        for (int e = tid; e < 128 * nr; e += NTH) {
            const int64_t i = row0 + e % 128;
            if (i < T.n) Bc[i + (int64_t)(e / 128) * ldb] = __builtin_nan("");
        }
    };
    int seen = 0;
    struct Piece {
        Raw<!FWD> r;
        TileRef R;
    } p0, p1, p2;
    auto start = [&](int k, Piece &p) {
        if (k < count) {
            p.R = ref(k);
            fetch_step(k, p.R, p.r);
        }
    };
    // step k with its piece in use, the one of step k + 2 sent for behind the values
    // just received: loads return in order, and a poll behind a piece on its way
    // from memory would wait for that first
    auto step = [&](int k, Piece &use, Piece &next) -> bool {
        if (count - k > NEAR && k >= seen) {
            if (tid == 0) s_word = wait_count(c, copy, k + 1);
            __syncthreads();
            seen = s_word;
            if (seen < 0) {
                give_up();
                return false;
            }
        }
        double *x = xs[k & 1];
        const unsigned long long *m = mc + (int64_t)(FWD ? k : first - k) * PER;
        constexpr int EPT = (PER + NTH - 1) / NTH;
        unsigned long long u[EPT];
#pragma unroll
        for (int j = 0; j < EPT; ++j)
            if (PER >= NTH || tid < PER) u[j] = ld_mail(m + tid + NTH * j);
#pragma unroll
        for (int j = 0; j < EPT; ++j)
            if (PER >= NTH || tid < PER) {
                const int e = tid + NTH * j;
                if (!receive(c, m + e, u[j])) s_late = 1;
                x[ONE ? e : (e % HB) * LDX + e / HB] = __longlong_as_double((long long)u[j]);
            }
        __syncthreads();
        if (s_late) {
            give_up();
            return false;
        }
        start(k + 2, next);
        if (!second || k + 1 < count) product(use.r, use.R, x);  // the last one: below
        return true;
    };
    start(0, p0);
    start(1, p1);
    for (int k = 0; k < count; k += 3) {
        if (!step(k, p0, p2)) return;
        if (k + 1 < count && !step(k + 1, p1, p0)) return;
        if (k + 2 < count && !step(k + 2, p2, p1)) return;
    }

    // the block between the halves, in flight while the first is solved
    Raw<!FWD> mid;
    if constexpr (FWD) {
        if (second) fetch(D, lr + wave * 16 + gi + (lr + (ONE ? 16 : 1) * gg) * b, (ONE ? 1 : 4) * b, mid);
    } else {
        if (second) fetch(D, lr + HB + 2 * gg + (lr + wave * 16 + gi) * b, mid);
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
                if (gg == 0) rs[0][w * 16 + gi] = 0.0 - acc.t[0];
            } else {
#pragma unroll
                for (int v = 0; v < 4; ++v) rs[gi][w * 16 + gg + 4 * v] = 0.0 - acc.t[v];
            }
        }
        __syncthreads();
        if (half == 0 && second && count > 0) {  // their last step, beside the solve of the first half
            const double *x = xs[1];
            if (count % 3 == 1) product(p0.r, p0.R, x);
            else if (count % 3 == 2) product(p1.r, p1.R, x);
            else product(p2.r, p2.R, x);
        }
        // two waves of the rows solved first (one for ONE), eight right-hand sides each
        const int sw = wave - (FWD ? 0 : WAVES / 2);
        constexpr int NQ = ONE ? 1 : 2;
        const int q0 = ONE ? 0 : sw * 8 + gg * 2;
        const bool solver = sw == 0 || (!ONE && sw == 1);
        double v[4][NQ];
        if (solver) {
            double d[4], rd[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                d[t] = dg[h * HB + 16 * t + gi];
                rd[t] = rg[h * HB + 16 * t + gi];
            }
            auto divide = [&]() {
                bool fits = plain;
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int q = 0; q < NQ; ++q) fits &= in_range(v[t][q]) || v[t][q] == 0.0;
                if (__all(fits)) {
#pragma unroll
                    for (int t = 0; t < 4; ++t)
#pragma unroll
                        for (int q = 0; q < NQ; ++q) v[t][q] = div_by(v[t][q], d[t], rd[t]);
                } else {
#pragma unroll
                    for (int t = 0; t < 4; ++t)
#pragma unroll
                        for (int q = 0; q < NQ; ++q) v[t][q] = v[t][q] / d[t];
                }
            };
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int q = 0; q < NQ; ++q) v[t][q] = rs[q0 + q][16 * t + gi];
            if (!FWD) divide();
            solve64<FWD, NQ>(v, ds[h], gi);
            if (FWD) divide();
            unsigned long long *m = mc + (row0 / HB + h) * PER + gi;
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int q = 0; q < NQ; ++q)
                    if (!ONE || gg == 0) {
                        st_mail(m + (q0 + q) * HB + 16 * t, v[t][q]);
                        xh[ONE ? 16 * t + gi : (16 * t + gi) * LDX + q0 + q] = v[t][q];
                    }
        }
        __syncthreads();
        if (solver) {
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
                    const int64_t i = row0 + h * HB + 16 * t + gi;
                    if (i < T.n && q0 + q < nr && (!ONE || gg == 0)) Bc[i + (int64_t)(q0 + q) * ldb] = v[t][q];
                }
        }
    }
    stores_done();
    __syncthreads();
    if (tid < NCOPY) raise_count(c.done + tid * STRIDE, count + 2);
}

// Right-hand sides per launch: 16 chunks share a launch, each with its own chain.
constexpr int MAXCHUNK = 16;

size_t solve_ctl_bytes() { return (size_t)2 * (32 + MAXCHUNK * NCOPY * STRIDE) * sizeof(int); }

// Places of one direction's mailbox for nr right-hand sides of a launch.
static int64_t solve_places(int64_t n, int nr)
{
    return (n + 127) / 128 * 128 * (nr == 1 ? 1 : NR * ((nr + NR - 1) / NR));
}

size_t solve_mail_bytes(int64_t n, int nrhs)
{
    return (size_t)solve_places(n, nrhs < MAXCHUNK * NR ? nrhs : MAXCHUNK * NR) * 2 * sizeof(double);
}

void launch_solve(const Tiles &T, double *B, int64_t ldb, int nrhs, int *ctl, double *mail, int *late, hipStream_t st)
{
    const int words = (int)(solve_ctl_bytes() / sizeof(int));
    const unsigned nblk = (unsigned)((T.n + 127) / 128);
    unsigned long long *mf = (unsigned long long *)mail;
    for (int j0 = 0; j0 < nrhs; j0 += MAXCHUNK * NR) {
        const int nr = nrhs - j0 < MAXCHUNK * NR ? nrhs - j0 : MAXCHUNK * NR;
        double *Bj = B + (int64_t)j0 * ldb;
        const unsigned chunks = (unsigned)((nr + NR - 1) / NR), grid = nblk * chunks;
        const int64_t places = solve_places(T.n, nr);
        int *bwd = ctl + words / 2;
        unsigned long long *mb = mf + places;
        const int64_t fill = (2 * places + 1023) / 1024;
        solve_reset_kernel<<<(unsigned)(fill < 16 ? 16 : fill > 2048 ? 2048 : fill), 256, 0, st>>>(ctl, words, mf, 2 * places);
        if (nr == 1) {
            solve_kernel<true, true><<<grid, NTH, 0, st>>>(T, Bj, ldb, nr, ctl, mf, late, WAIT_TICKS);
            solve_kernel<false, true><<<grid, NTH, 0, st>>>(T, Bj, ldb, nr, bwd, mb, late, WAIT_TICKS);
        } else {
            solve_kernel<true, false><<<grid, NTH, 0, st>>>(T, Bj, ldb, nr, ctl, mf, late, WAIT_TICKS);
            solve_kernel<false, false><<<grid, NTH, 0, st>>>(T, Bj, ldb, nr, bwd, mb, late, WAIT_TICKS);
        }
    }
}

}  // namespace mpc
