// predict_impl.h -- prediction with the ensemble held in LDS (predict.hip).
#pragma once

#include "common.h"

namespace gbt {

// An ensemble in the compact form the kernels read, on the device.
struct LdsTrees {
    const uint32_t *words = nullptr;  // per tree: 2^depth - 1 splits of two words, then 2^depth leaf values
    const int4 *chunks = nullptr;     // {first word, words, first tree, end tree} of trees staged together
    const int32_t *depth = nullptr;   // depth of each tree
    int32_t n_chunks = 0;
    int32_t chunk_words = 0;          // words of the largest chunk
    std::vector<char> host;           // what the upload reads, unless that is host_io's buffer
};

// Rows per block for the ensemble over n_rows rows of row_words 32-bit words
// (binned: of symbols), or 0 when it does not fit the LDS (trees deeper than
// 11, rows above about 500 words) or its steps are too few to pay for staging
// the rows: then the trees are walked in global memory.
int32_t lds_predict_rows(const gbt_tree *trees, int32_t n_trees, int64_t n_rows, int32_t row_words, bool binned);

// Compacts the trees and uploads them.  w > 0: splits of binned rows with
// w-bit symbols; w = 0: splits of raw values.  *ok is false (and nothing is
// uploaded) when a split names no column of the n_cols.  The copy reads
// out->host or the pinned buffer of host_io: the stream is to be synchronized
// before the one is destroyed or the other used again.
gbt_status lds_upload_trees(gbt_ctx *c, const gbt_tree *trees, int32_t n_trees, int32_t w, int32_t n_cols,
                            LdsTrees *out, bool *ok);

gbt_status lds_predict_raw(gbt_ctx *c, const LdsTrees &t, const float *X, int64_t n, int32_t m, int64_t ld, float base,
                           int32_t block_rows, float *out);
gbt_status lds_predict_binned(gbt_ctx *c, const LdsTrees &t, const uint32_t *words, int64_t n, const Geo &geo,
                              float base, int32_t block_rows, float *out);

}  // namespace gbt
