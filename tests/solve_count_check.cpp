// CPU check of the solve's count of finished blocks (csrc/k_solve.hip), run by
// tests/test_host_logic.py: the chain's workgroups publish in an order given on
// the command line; prints the count after each.
#include <cstdio>
#include <cstdlib>

#include "../paper_2408_04440_amd/csrc/k_solve.hip"

int main(int argc, char **argv)
{
    int done = 0;
    for (int i = 1; i < argc; ++i) {
        mpc::raise_count(&done, 2 * atoi(argv[i]) + 2);  // as place argv[i] of the chain
        printf("%d ", done);
    }
    return 0;
}
