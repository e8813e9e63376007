// Emulation draws Y = L Z from the stored factor (Sec. III.B), with the
// Philox4x32-10 / Box-Muller normal generator.
#include <type_traits>

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
// One BM x BN block of Y per workgroup of four waves: rows of tile row I,
// columns of draws; sum over K <= I of L_IK Z_K on the FP32 MFMA, each stored
// tile widened (exactly, or rounded to FP32 for FP64 tiles) on its way into LDS.
// What bounds it: the FP32 MFMA for many draws (64 x 64 outputs a wave, 16
// products per eight LDS reads), the factor's bytes for few.  Raw codes of the
// next K slice stay in registers while the current one is multiplied and are
// converted only when staged, by a loop per class; every class takes the same
// 16-byte loads, so that no branch, and no wait, stands between them.  The last
// tile rows, with the most tiles to walk, take the first blocks.  (Four waves of
// 64 x 64 in place of sixteen of 32 x 32, N = 16,384, 1000 draws: 4.92 -> 2.97 ms;
// an order in which the strips of equal length met on the same compute units took
// 5.2 ms.  Without class branches between the loads and conversions: 2.97 -> 2.88
// ms, 93 TFLOP/s; one draw 0.51 -> 0.46 ms, 2.3 TB/s of the factor; N = 32,768
// under the norm rule, 100 draws 2.85 -> 2.48, 1000 draws 13.6 -> 11.7.)
constexpr int ANT = 256;

// Two consecutive values of a stored tile, byte the offset of the first within it.
template <int CLS> __device__ inline float2 widen32(ulonglong2 v, int byte, int lo16, int t)
{
    if (CLS == P64)
        return make_float2((float)__longlong_as_double((long long)v.x), (float)__longlong_as_double((long long)v.y));
    const uint64_t u = pair_codes(v, byte);
    const uint32_t w = (uint32_t)u;
    if (CLS == P32) return make_float2(__uint_as_float(w), __uint_as_float((uint32_t)(u >> 32)));
    constexpr int BITS = CLS == P16 ? 16 : 8;
    constexpr uint32_t MASK = (1u << BITS) - 1;
    return make_float2((float)decode_class(w & MASK, CLS, lo16, t), (float)decode_class((w >> BITS) & MASK, CLS, lo16, t));
}

template <int BM, int BN, int AK>
__global__ __launch_bounds__(ANT) void lower_apply_kernel(Tiles T, const float *__restrict__ Z, int64_t ldz, float *Y,
                                                          int64_t ldy, int ndraws)
{
    constexpr int WM = BM == 32 && BN >= 64 ? 1 : 2, WN = BN >= 64 ? 4 / WM : 1;  // waves along rows and draws (the rest only load)
    constexpr int MB = BM / WM / 16, NB = BN / WN / 16;
    constexpr int LDA = BM + 16, LDB = BN + 4;
    constexpr int APER = AK * BM / ANT / 2, BPER = AK * BN / ANT;  // A: row pairs, B: K elements per thread
    constexpr int ACOL = 2 * ANT / BM, BCOL = ANT / AK;            // columns of A, draws of B per round
    __shared__ float As[2][AK][LDA], Bs[2][AK][LDB];
    const int b = T.b, nsub = b / BM;
    // consecutive workgroups go to the XCDs in turn: the blocks of one row strip
    // follow each other on one XCD, whose L2 then serves its tiles to all of them
    const int ny = (ndraws + BN - 1) / BN, xcd = blockIdx.x % 8, idx = blockIdx.x / 8;
    const int strip = idx / ny * 8 + xcd;
    if (strip >= T.nt * nsub) return;
    const int I = T.nt - 1 - strip / nsub, tm = nsub - 1 - strip % nsub;
    const int s0 = idx % ny * BN;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave % WM, wn = wave / WM, gi = lane & 15, gg = lane >> 4;
    float4_t acc[MB][NB];
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int n = 0; n < NB; ++n) acc[m][n] = (float4_t){0.f, 0.f, 0.f, 0.f};
    const int nkt = b / AK, total = (I + 1) * nkt;
    // slice q: tile q / nkt of the row, columns (q % nkt) * AK
    ulonglong2 ra[APER];
    float rb[BPER];
    int ca = 0, ta = 0, next = 0;
    const int r2 = 2 * (tid % (BM / 2)), c0 = tid / (BM / 2);  // A: rows r2, r2 + 1 of columns c0 + ACOL c
    const int kb = tid % AK, n0 = tid / AK;                    // B: K element kb of draws n0 + BCOL c
    const float *zb = Z + (int64_t)(s0 + n0) * ldz + kb;
    const bool whole = s0 + BN <= ndraws;
    auto class_at = [&](int K) { return (I == K) ? (int)P64 : (int)T.map[I + (int64_t)K * T.nt]; };
    auto gload = [&](int q) {
        const int K = q / nkt, k0 = (q - K * nkt) * AK;
        ca = __builtin_amdgcn_readfirstlane(next);  // read a slice ahead
        next = class_at(min(q + 1, total - 1) / nkt);
        ta = T.tscale[I + (int64_t)K * T.nt];
        const char *sa = T.slots + tile_index(I, K) * T.slot_bytes;
        const int off = tm * BM + r2 + (k0 + c0) * b, sh = class_shift(ca);  // within one tile: below b * b
#pragma unroll
        for (int c = 0; c < APER; ++c) ra[c] = load_pair16(sa, (off + ACOL * c * b) << sh);
        const int64_t zk = (int64_t)K * b + k0;
        if (whole && zk + AK <= T.n) {
#pragma unroll
            for (int c = 0; c < BPER; ++c) rb[c] = zb[zk + (int64_t)(BCOL * c) * ldz];
        } else {  // absent draws repeat the last one (their columns of Y are not written)
            const int64_t zr = min(zk + kb, T.n - 1);
#pragma unroll
            for (int c = 0; c < BPER; ++c) {
                const float v = Z[zr + (int64_t)min(s0 + n0 + BCOL * c, ndraws - 1) * ldz];
                rb[c] = zk + kb < T.n ? v : 0.0f;
            }
        }
    };
    auto astore = [&](auto cls, int buf) {  // a loop per class: no branch between its conversions
        constexpr int CLS = decltype(cls)::value;
#pragma unroll
        for (int c = 0; c < APER; ++c)  // strips and columns start at multiples of 32 values
            *(float2 *)&As[buf][c0 + ACOL * c][r2] = widen32<CLS>(ra[c], r2 << class_shift(CLS), T.lo16, ta);
    };
    auto sstore = [&](int buf) {
        switch (ca) {
        case P64: astore(std::integral_constant<int, P64>{}, buf); break;
        case P32: astore(std::integral_constant<int, P32>{}, buf); break;
        case P16: astore(std::integral_constant<int, P16>{}, buf); break;
        default: astore(std::integral_constant<int, P8>{}, buf); break;
        }
#pragma unroll
        for (int c = 0; c < BPER; ++c) Bs[buf][kb][n0 + BCOL * c] = rb[c];
    };
    next = class_at(0);
    gload(0);
    sstore(0);
    __syncthreads();
    for (int q = 0; q < total; ++q) {
        const int cur = q & 1;
        if (q + 1 < total) gload(q + 1);
        if (WM * WN == 4 || wave < WM * WN)
#pragma unroll
        for (int s = 0; s < AK / 4; ++s) {
            float fa[MB], fb[NB];
#pragma unroll
            for (int m = 0; m < MB; ++m) fa[m] = As[cur][s * 4 + gg][(wm * MB + m) * 16 + gi];
#pragma unroll
            for (int n = 0; n < NB; ++n) fb[n] = Bs[cur][s * 4 + gg][(wn * NB + n) * 16 + gi];
#pragma unroll
            for (int m = 0; m < MB; ++m)
#pragma unroll
                for (int n = 0; n < NB; ++n)
                    acc[m][n] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[m], fb[n], acc[m][n], 0, 0, 0);
        }
        if (q + 1 < total) sstore(cur ^ 1);
        __syncthreads();
    }
    if (WM * WN < 4 && wave >= WM * WN) return;
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int n = 0; n < NB; ++n)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int64_t i = (int64_t)I * b + tm * BM + (wm * MB + m) * 16 + 4 * gg + v;
                const int s = s0 + (wn * NB + n) * 16 + gi;
                if (i < T.n && s < ndraws) Y[i + (int64_t)s * ldy] = acc[m][n][v];
            }
}

template <int BM, int BN, int AK>
static void launch_apply(const Tiles &T, const float *Z, int64_t ldz, float *Y, int64_t ldy, int ndraws, hipStream_t st)
{
    const unsigned strips = (unsigned)(T.nt * (T.b / BM)), grid = (strips + 7) / 8 * 8 * ((ndraws + BN - 1) / BN);
    lower_apply_kernel<BM, BN, AK><<<grid, ANT, 0, st>>>(T, Z, ldz, Y, ldy, ndraws);
}

// Draws per block: 128, and for few draws the smallest of 16 and 64 that holds
// them, so that no products are spent on absent columns.  A strip of 128 rows
// walks up to n columns in sequence; where they are too few to fill the GPU
// twice over and even out their lengths (fewer than 1024 workgroups), strips of
// 32 rows do (N = 32,400, 100 draws: 5.4 against 2.5 ms; N = 16,384, 512: 2.0
// against 1.8).
void launch_lower_apply(const Tiles &T, const float *Z, int64_t ldz, float *Y, int64_t ldy, int ndraws, hipStream_t st)
{
    if (ndraws <= 16) launch_apply<32, 16, 64>(T, Z, ldz, Y, ldy, ndraws, st);
    else if (ndraws <= 64) launch_apply<32, 64, 64>(T, Z, ldz, Y, ldy, ndraws, st);
    else if ((int64_t)T.nt * (T.b / 128) * ((ndraws + 127) / 128) < 1024)
        launch_apply<32, 128, 32>(T, Z, ldz, Y, ldy, ndraws, st);
    else launch_apply<128, 128, 32>(T, Z, ldz, Y, ldy, ndraws, st);
}

}  // namespace mpc
