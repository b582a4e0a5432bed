// The host side of the kernels' index and key arithmetic, for test_device_math.py.
#include "common.h"

extern "C" {
long long inplace_row(int run, int run_rows, int row_of_run) { return cmp::inplace_row(run, run_rows, row_of_run); }
int inplace_runs(int rows, int run_rows) { return cmp::inplace_runs(rows, run_rows); }
int inplace_moves(int tok, long long j, int n) { return cmp::inplace_moves(tok, j, n); }
void head_chunks(int n, int per_block, int *blocks, int *chunk) {
  *blocks = cmp::blocks_per_head(n, per_block, 4);
  *chunk = cmp::chunk_of(n, per_block, 4);
}
int chunk_tokens(int begin, int chunk, int n) { return cmp::chunk_tokens(begin, chunk, n); }
int quad_at(int begin, int at, int tokens) { return cmp::quad_base(begin, tokens) + cmp::quad_from_base(at, tokens); }
int inplace_late_token(void) { return cmp::INPLACE_LATE; }
int sample_lines(void) { return cmp::SAMPLE_LINES; }
int sample_line(int g, int lines) { return cmp::sample_line(g, lines); }
int score_bin(unsigned key) { return cmp::score_bin(key); }
int bin_bits(int bin, int fine, unsigned *lo) {
  const cmp::BinKeys k = cmp::bin_keys(bin, fine != 0);
  *lo = k.lo;
  return k.bits;
}
}
