// The report of a solve whose wait runs out, run by tests/test_gpu_solve_wait.py:
// the solve's kernels are launched without the first place of their chain (its
// ticket is taken here), under a limit of 10 ms, so that every other place waits
// for values that nobody writes, gives up and ends.  Includes the two sources for
// their internals; linked with the library's other objects.
#include "../paper_2408_04440_amd/csrc/k_solve.hip"
#include "../paper_2408_04440_amd/csrc/mpchol.cpp"

#include <cstring>

#define CHECK(c)                                                          \
    do {                                                                  \
        if (!(c)) {                                                       \
            fprintf(stderr, "line %d: %s failed: %s\n", __LINE__, #c, mpchol_last_error()); \
            exit(1);                                                      \
        }                                                                 \
    } while (0)

// One direction with place 0 left out; rows of the places that waited must be NaN, the others as they were.
template <bool FWD, bool ONE> static void without_the_first(mpchol_t h, int nrhs, double *B, const std::vector<double> &hb)
{
    const int64_t n = h->n;
    const unsigned nblk = (unsigned)((n + 127) / 128);
    const int words = (int)(solve_ctl_bytes() / sizeof(int));
    const int64_t places = (int64_t)nblk * 128 * (ONE ? 1 : 16);
    const unsigned taken = 1;
    CHECK(hipMemcpy(B, hb.data(), hb.size() * 8, hipMemcpyHostToDevice) == hipSuccess);
    solve_reset_kernel<<<16, 256, 0, h->st>>>(h->d_solve, words, (unsigned long long *)h->p64, places);
    CHECK(hipStreamSynchronize(h->st) == hipSuccess);
    CHECK(hipMemcpy(h->d_solve, &taken, 4, hipMemcpyHostToDevice) == hipSuccess);
    CHECK(*h->late() == 0);
    solve_kernel<FWD, ONE><<<nblk - 1, 512, 0, h->st>>>(h->tiles(), B, n, nrhs, h->d_solve, (unsigned long long *)h->p64,
                                                        h->late(), 1000000);
    CHECK(hipStreamSynchronize(h->st) == hipSuccess);
    std::vector<double> x(hb.size());
    CHECK(hipMemcpy(x.data(), B, x.size() * 8, hipMemcpyDeviceToHost) == hipSuccess);
    const int64_t lo = FWD ? 0 : ((int64_t)nblk - 1) * 128, hi = FWD ? 128 : n;  // rows of the place left out
    for (int q = 0; q < nrhs; ++q)
        for (int64_t i = 0; i < n; ++i)
            CHECK((i >= lo && i < hi) ? x[i + q * n] == hb[i + q * n] : std::isnan(x[i + q * n]));
    CHECK(*h->late() == 1);
}

int main()
{
    const int64_t n = 1000;
    std::vector<double> sigma(n), x(n), hb(n * 3);
    for (int64_t i = 0; i < n; ++i) sigma[i] = 1.0 + 0.1 * std::sin((double)i), x[i] = (double)i;
    for (size_t i = 0; i < hb.size(); ++i) hb[i] = std::cos((double)i);
    mpchol_t h = nullptr;
    CHECK(mpchol_create(&h, n, 256, nullptr) == MPCHOL_OK);
    CHECK(mpchol_set_generator(h, sigma.data(), x.data(), 5.0, 1e-8) == MPCHOL_OK);
    CHECK(mpchol_precision_map(h, MPCHOL_RULE_FP64, 1e-9, nullptr, nullptr) == MPCHOL_OK);
    CHECK(mpchol_factor(h, nullptr) == MPCHOL_OK);
    double *B = nullptr, want = 0, ld = 0, be = 0;
    float *Y = nullptr;
    CHECK(hipMalloc(&B, hb.size() * 8) == hipSuccess && hipMalloc(&Y, n * 4) == hipSuccess);
    CHECK(mpchol_logdet(h, &want) == MPCHOL_OK);
    mpchol_stats st;
    std::vector<int32_t> ts(h->nt * h->nt);
    std::vector<double> A(n * n, 1.0);
    for (int c = 0; c < 7; ++c) {
        printf("case %d\n", c);
        fflush(stdout);
        if (c % 4 == 0) without_the_first<true, true>(h, 1, B, std::vector<double>(hb.begin(), hb.begin() + n));
        else if (c % 4 == 1) without_the_first<false, true>(h, 1, B, std::vector<double>(hb.begin(), hb.begin() + n));
        else if (c % 4 == 2) without_the_first<true, false>(h, 3, B, hb);
        else without_the_first<false, false>(h, 3, B, hb);
        // each of the calls that synchronize reports it, and only once
        auto call = [&]() {
            switch (c) {
            case 0: return mpchol_logdet(h, &ld);
            case 1: return mpchol_get_stats(h, &st);
            case 2: return mpchol_get_tile_scales(h, ts.data());
            case 3: return mpchol_backward_error(h, &be, nullptr);
            case 4: return mpchol_backward_error_estimate(h, 1, 7, &be);
            case 5: return mpchol_backward_error_matrix(h, A.data(), n, 0, &be, nullptr);
            default: return mpchol_sample(h, 1, 3, Y, n);
            }
        };
        CHECK(call() == MPCHOL_EHIP);
        CHECK(std::strstr(mpchol_last_error(), "mpchol_solve") != nullptr);
        CHECK(call() == MPCHOL_OK);
        CHECK(mpchol_solve(h, 3, B, n) == MPCHOL_OK);  // whatever was left behind, the next solve is whole
        CHECK(mpchol_logdet(h, &ld) == MPCHOL_OK && ld == want);
    }
    CHECK(hipFree(B) == hipSuccess && hipFree(Y) == hipSuccess);
    CHECK(mpchol_destroy(h) == MPCHOL_OK);
    printf("ok\n");
    return 0;
}
