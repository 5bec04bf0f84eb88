// Rows that a workgroup of the append and gather kernels copies, for test_copy_grid.py.
#include "kargs.h"

extern "C" uint32_t rows_per_block(uint32_t row_elems) { return cp::copy_rows_per_block(row_elems); }
extern "C" int threads_per_block() { return cp::kCopyThreads; }
