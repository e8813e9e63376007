// Emulation draws Y = L Z from the stored factor (Sec. III.B), with the
// Philox4x32-10 / Box-Muller normal generator.
#include "common.h"
#include "launch.h"

namespace mpc {

// ---------------------------------------------------------------- normal draws
// Philox4x32-10 (Salmon et al., SC'11): 10 rounds of the multiply/xor
// bijection with key schedule increments W0, W1.
__device__ inline void philox4x32_10(uint32_t &c0, uint32_t &c1, uint32_t &c2, uint32_t &c3, uint32_t k0, uint32_t k1)
{
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        uint32_t lo0 = 0xD2511F53u * c0, hi0 = __umulhi(0xD2511F53u, c0);
        uint32_t lo1 = 0xCD9E8D57u * c2, hi1 = __umulhi(0xCD9E8D57u, c2);
        uint32_t n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
        c0 = n0;
        c1 = lo1;
        c2 = n2;
        c3 = lo0;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
}

// Draw e (e = i + d*n, the column-major index of an n x ndraws array) comes
// from counter block e/4, output e%4: uniforms ((x >> 8) + 1) 2^-24 in (0,1],
// Box-Muller on (u0,u1) and (u2,u3) in FP32.  A launch writes the draws
// e0 <= e < e0 + count (e0 a multiple of n: whole columns starting at column
// e0/n) to Z with the column index taken relative to e0/n; each value depends
// only on e, so a range gives the same values as the whole sequence.
__global__ __launch_bounds__(256) void normal_kernel(uint64_t seed, int64_t e0, int64_t count, int64_t n, float *Z,
                                                     int64_t ldz, uint32_t *raw)
{
    const int64_t blk = e0 / 4 + (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (blk * 4 >= e0 + count) return;
    uint32_t c0 = (uint32_t)blk, c1 = (uint32_t)((uint64_t)blk >> 32), c2 = 0, c3 = 0;
    philox4x32_10(c0, c1, c2, c3, (uint32_t)seed, (uint32_t)(seed >> 32));
    uint32_t o[4] = {c0, c1, c2, c3};
    float u[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) u[q] = (float)((o[q] >> 8) + 1u) * 5.9604644775390625e-8f;  // 2^-24
    const float twopi = 6.28318530717958647692f;
    float r0 = sqrtf(-2.0f * logf(u[0])), r1 = sqrtf(-2.0f * logf(u[2]));
    float s0, k0, s1, k1;
    sincosf(twopi * u[1], &s0, &k0);
    sincosf(twopi * u[3], &s1, &k1);
    float v[4] = {r0 * k0, r0 * s0, r1 * k1, r1 * s1};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int64_t e = blk * 4 + q;
        if (e < e0) continue;
        if (e >= e0 + count) break;
        const int64_t l = e - e0;
        if (Z) Z[(l % n) + (l / n) * ldz] = v[q];
        if (raw) raw[l] = o[q];
    }
}

static void launch_normal(uint64_t seed, int64_t e0, int64_t count, int64_t n, float *Z, int64_t ldz, uint32_t *raw,
                          hipStream_t st)
{
    const int64_t nb = (e0 + count + 3) / 4 - e0 / 4;  // counter blocks touched
    normal_kernel<<<(unsigned)((nb + 255) / 256), 256, 0, st>>>(seed, e0, count, n, Z, ldz, raw);
}

void launch_normal_draws(uint64_t seed, int64_t count, float *z, uint32_t *raw, hipStream_t st)
{
    launch_normal(seed, 0, count, count, z, count, raw, st);
}

void launch_normal_matrix(uint64_t seed, int64_t n, int ndraws, float *Z, int64_t ldz, hipStream_t st)
{
    launch_normal(seed, 0, n * ndraws, n, Z, ldz, nullptr, st);
}

void launch_normal_columns(uint64_t seed, int64_t n, int64_t d0, int nd, float *Z, int64_t ldz, hipStream_t st)
{
    launch_normal(seed, d0 * n, n * nd, n, Z, ldz, nullptr, st);
}

// ---------------------------------------------------------------- Y = L Z
// One 128 x 128 block of Y per workgroup of 16 waves (32 x 32 each): rows of
// tile row I, columns of draws; sum over K <= I of L_IK Z_K with FP32 MFMA,
// each stored tile widened (exactly, or rounded to FP32 for FP64 tiles) on its
// way into LDS.  The last tile rows, with the most tiles to walk, take the
// first blocks.
constexpr int SB = 128, SK = 16, SLD = SB + 4, SW = 4, SNT = 64 * SW * SW, SPER = SK * SB / SNT;

__global__ __launch_bounds__(SNT) void lower_apply_kernel(Tiles T, const float *Z, int64_t ldz, float *Y, int64_t ldy,
                                                          int ndraws)
{
    __shared__ float As[2][SK][SLD], Bs[2][SK][SLD];
    const int b = T.b, nsub = b / SB;
    const int I = T.nt - 1 - (int)(blockIdx.x / nsub), tm = blockIdx.x % nsub;
    const int s0 = blockIdx.y * SB;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave % SW, wn = wave / SW, gi = lane & 15, gg = lane >> 4;
    constexpr int WT = SB / SW;
    float4_t acc[2][2];
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int n = 0; n < 2; ++n) acc[m][n] = (float4_t){0.f, 0.f, 0.f, 0.f};
    const int nkt = b / SK;
    float ra[SPER], rb[SPER];
    for (int K = 0; K <= I; ++K) {
        const int ca = (I == K) ? P64 : T.map[I + (int64_t)K * T.nt];
        const int ta = T.tscale[I + (int64_t)K * T.nt];
        const char *sa = T.slots + tile_index(I, K) * T.slot_bytes;
        auto gload = [&](int kt) {
#pragma unroll
            for (int c = 0; c < SPER; ++c) {
                int e = tid + SNT * c;
                int r = e % SB, col = e / SB;
                ra[c] = (float)load_stored(sa, ca, T.lo16, ta, (int64_t)(tm * SB + r) + (int64_t)(kt * SK + col) * b);
                int kk = e % SK, s = e / SK;
                int64_t zr = (int64_t)K * b + kt * SK + kk;
                rb[c] = (zr < T.n && s0 + s < ndraws) ? Z[zr + (int64_t)(s0 + s) * ldz] : 0.0f;
            }
        };
        auto sstore = [&](int buf) {
#pragma unroll
            for (int c = 0; c < SPER; ++c) {
                int e = tid + SNT * c;
                As[buf][e / SB][e % SB] = ra[c];
                Bs[buf][e % SK][e / SK] = rb[c];
            }
        };
        gload(0);
        sstore(0);
        __syncthreads();
        for (int kt = 0; kt < nkt; ++kt) {
            const int cur = kt & 1;
            if (kt + 1 < nkt) gload(kt + 1);
#pragma unroll
            for (int s = 0; s < SK / 4; ++s) {
                float fa[2], fb[2];
#pragma unroll
                for (int m = 0; m < 2; ++m) fa[m] = As[cur][s * 4 + gg][wm * WT + m * 16 + gi];
#pragma unroll
                for (int n = 0; n < 2; ++n) fb[n] = Bs[cur][s * 4 + gg][wn * WT + n * 16 + gi];
#pragma unroll
                for (int m = 0; m < 2; ++m)
#pragma unroll
                    for (int n = 0; n < 2; ++n)
                        acc[m][n] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[m], fb[n], acc[m][n], 0, 0, 0);
            }
            if (kt + 1 < nkt) sstore(cur ^ 1);
            __syncthreads();
        }
    }
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int n = 0; n < 2; ++n)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                int64_t i = (int64_t)I * b + tm * SB + wm * WT + m * 16 + 4 * gg + v;
                int s = s0 + wn * WT + n * 16 + gi;
                if (i < T.n && s < ndraws) Y[i + (int64_t)s * ldy] = acc[m][n][v];
            }
}

void launch_lower_apply(const Tiles &T, const float *Z, int64_t ldz, float *Y, int64_t ldy, int ndraws, hipStream_t st)
{
    dim3 grid(T.nt * (T.b / SB), (ndraws + SB - 1) / SB);
    lower_apply_kernel<<<grid, SNT, 0, st>>>(T, Z, ldz, Y, ldy, ndraws);
}

}  // namespace mpc
