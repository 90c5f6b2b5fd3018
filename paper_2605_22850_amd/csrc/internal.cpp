// What the tests ask of the library's dispatch rules (no GPU needed).  Not
// part of the C ABI.
#include "common.hpp"

using namespace oc;

extern "C" {

// Whether the few-row kernels take a product, and how many ranges they split
// its K into.
int oc_internal_gemm_rows(int64_t M, int64_t K, int64_t N, int has_workspace, int64_t *n_split) {
    const bool ours = gemm_rows_applies(M, K, N, has_workspace != 0);
    *n_split = ours ? gemm_rows_splits(M, K, N) : 0;
    return ours;
}

}  // extern "C"
