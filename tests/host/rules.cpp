// rules.cpp -- the host's rules on sizes (som_rules.h), for the tests (fixture `rules`).
#include "../../paper_2608_24067_amd/csrc/som_internal.h"

extern "C" {
int64_t group_tiles(int64_t nt, int64_t strips, int32_t ta, int32_t f16)
{
    return som::sweep_group_tiles(nt, strips, ta, f16 != 0);
}
int32_t rows_direct(int64_t N, int64_t M, int64_t nnz, int32_t ta, int32_t f16)
{
    return som::rows_direct(N, M, nnz, ta, f16 != 0);
}
int32_t regroups(int64_t N, int64_t M, int64_t nnz, int32_t ta) { return som::regroup_pays(N, M, nnz, ta); }
int64_t strips(int64_t M, int32_t ta) { return som::n_strips(M, ta); }
}
