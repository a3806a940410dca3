// Prints tc::hot_width for tiles read from stdin, one a line:
// lds_stage n_cu lds_floats n_cols col_begin col_end nnz hot_nnz long items
#include <cstdio>

#include "tc_tile.h"

int main() {
  long long stage, n_cu, lds, n_cols, cb, ce, nnz, hot, longest, items;
  while (std::scanf("%lld %lld %lld %lld %lld %lld %lld %lld %lld %lld", &stage, &n_cu, &lds, &n_cols, &cb, &ce, &nnz,
                    &hot, &longest, &items) == 10) {
    tc_handle h;
    h.lds_tiles = (int32_t)stage + 1;
    h.n_cu = (int)n_cu;
    h.lds_floats = lds;
    h.n_cols = n_cols;
    h.tile_col_begin = {cb};
    h.tile_col_end = {ce};
    h.tile_nnz = {nnz};
    h.tile_hot_nnz = {hot};
    h.tile_long = {longest};
    std::printf("%lld\n", (long long)tc::hot_width(&h, 0, items));
  }
}
