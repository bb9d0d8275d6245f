// predict.hip -- Eq. 1 prediction of raw dense rows and of dense binned rows
// with rows and trees in LDS.
//
// A block stages its rows once and the ensemble a chunk of trees at a time.
// A tree is compact: two words per split in heap order (the feature with its
// default direction, the threshold) and the values of its 2^D bottom places;
// the value of a leaf above the bottom fills every place below it, so a walk
// takes exactly D steps with no test for a leaf.  A lane owns a row and walks
// four trees of one depth at once (a step is two dependent LDS reads, the
// split and the row's value: four chains hide most of their latency), then
// adds their leaves in tree order, which keeps the float sum's order.
//
// The walk is bound by the LDS: 1 M rows x 28 features through 100 trees of
// depth 8 (800 M steps) take 0.48 ms, against 7.9 ms with one lane per row
// reading 48-byte nodes and the row from global memory.
#include "predict_impl.h"

#include <algorithm>
#include <cstring>

namespace gbt {

namespace {

constexpr int kMaxDepth = 11;               // 24.6 KB of one tree
constexpr int32_t kChunkWords = 4096;       // 16 KB of trees per chunk, or one larger tree
constexpr size_t kLdsRows256 = 80 << 10;    // LDS up to which two blocks of 256 rows share a CU
constexpr size_t kLdsRows64 = 150 << 10;
constexpr size_t kPinnedTrees = 4 << 20;     // bytes of compact trees uploaded from pinned memory
constexpr int kPinnedAfter = 16;            // calls from which a context allocates it for them
constexpr int64_t kFewRows = 64 * 512;      // up to here blocks of 64 rows use more CUs

int32_t tree_depth(const gbt_tree &t)
{
    int32_t d = 0;
    while (((2 << d) - 1) < t.n_nodes) ++d;
    return d;
}

int32_t tree_words(int32_t depth) { return ((3 << depth) - 2 + 3) / 4 * 4; }

int32_t row_pitch(int32_t row_words) { return (row_words + 1) | 1; }  // odd, with a word after the last one

struct RawStep {
    // bit 31 of x: missing goes left; the rest: the feature
    __device__ static bool left(uint2 nd, const uint32_t *row, uint32_t, uint32_t)
    {
        const float v = __uint_as_float(row[nd.x & 0x7fffffffu]);
        return v <= __uint_as_float(nd.y) || (v != v && (nd.x >> 31));
    }
};

struct BinStep {
    // x: the symbol's first bit; y: 2 * split_bin + (missing goes left)
    __device__ static bool left(uint2 nd, const uint32_t *row, uint32_t mask, uint32_t null_sym)
    {
        const uint32_t k = nd.x >> 5;
        const uint32_t sym = __builtin_amdgcn_alignbit(row[k + 1], row[k], nd.x & 31u) & mask;
        return sym == null_sym ? (nd.y & 1u) != 0 : sym < (nd.y >> 1);
    }
};

template <typename Step, int kU>
__device__ inline void walk(const uint32_t *tree, int32_t words, int32_t depth, const uint32_t *row, uint32_t mask,
                            uint32_t null_sym, float *acc)
{
    int32_t id[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) id[u] = 0;
    for (int32_t d = 0; d < depth; ++d) {
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const uint2 nd = *(const uint2 *)(tree + u * words + 2 * id[u]);
            id[u] = 2 * id[u] + (Step::left(nd, row, mask, null_sym) ? 1 : 2);
        }
    }
    // the bottom places follow the splits: place p at word 2 (2^D - 1) + p
    const int32_t last = (1 << depth) - 1;
#pragma unroll
    for (int u = 0; u < kU; ++u) *acc = *acc + __uint_as_float(tree[u * words + last + id[u]]);
}

template <typename Step>
__device__ inline void predict_rows(const uint32_t *__restrict__ words, const int4 *__restrict__ chunks,
                                    const int32_t *__restrict__ depth, int32_t n_chunks, uint32_t *tree_lds,
                                    const uint32_t *row, bool mine, uint32_t mask, uint32_t null_sym, float *acc)
{
    for (int32_t k = 0; k < n_chunks; ++k) {
        const int4 ch = chunks[k];
        __syncthreads();  // the chunk before is walked (and the rows are staged)
        const uint4 *src = (const uint4 *)(words + ch.x);
#pragma unroll 4
        for (int32_t i = threadIdx.x; i < ch.y / 4; i += (int32_t)blockDim.x) ((uint4 *)tree_lds)[i] = src[i];
        __syncthreads();
        if (!mine) continue;
        const uint32_t *t = tree_lds;
        int32_t i = ch.z;
        while (i < ch.w) {
            const int32_t d = depth[i], n = ((3 << d) - 2 + 3) / 4 * 4;
            if (i + 3 < ch.w && depth[i + 1] == d && depth[i + 2] == d && depth[i + 3] == d) {
                walk<Step, 4>(t, n, d, row, mask, null_sym, acc);
                t += 4 * n;
                i += 4;
            } else {
                walk<Step, 1>(t, n, d, row, mask, null_sym, acc);
                t += n;
                ++i;
            }
        }
    }
}

template <int kR>
__global__ void __launch_bounds__(kR)
    k_predict_raw_lds(const float *__restrict__ X, int64_t n, int32_t m, int64_t ld, uint32_t m_inv,
                      const uint32_t *__restrict__ words, const int4 *__restrict__ chunks,
                      const int32_t *__restrict__ depth, int32_t n_chunks, int32_t chunk_words, float base,
                      float *__restrict__ out)
{
    extern __shared__ __align__(16) uint32_t predict_lds[];
    uint32_t *rows = predict_lds + chunk_words;
    const int64_t r0 = (int64_t)blockIdx.x * kR;
    const int32_t nr = (int32_t)(n - r0 < kR ? n - r0 : kR);
    const int32_t pitch = (m + 1) | 1;
#pragma unroll 8
    for (uint32_t e = threadIdx.x; e < (uint32_t)(nr * m); e += kR) {
        const uint32_t r = m == 1 ? e : __umulhi(e, m_inv), c = e - r * (uint32_t)m;  // e / m, e % m
        rows[r * pitch + c] = __float_as_uint(X[(r0 + r) * ld + c]);
    }
    float acc = base;
    const bool mine = (int32_t)threadIdx.x < nr;
    predict_rows<RawStep>(words, chunks, depth, n_chunks, predict_lds, rows + threadIdx.x * pitch, mine, 0u, 0u, &acc);
    if (mine) out[r0 + threadIdx.x] = acc;
}

template <int kR>
__global__ void __launch_bounds__(kR)
    k_predict_bin_lds(const uint32_t *__restrict__ page, int64_t n, Geo geo, uint32_t q_inv,
                      const uint32_t *__restrict__ words, const int4 *__restrict__ chunks,
                      const int32_t *__restrict__ depth, int32_t n_chunks, int32_t chunk_words, float base,
                      float *__restrict__ out)
{
    extern __shared__ __align__(16) uint32_t predict_lds[];
    uint32_t *rows = predict_lds + chunk_words;
    const int64_t r0 = (int64_t)blockIdx.x * kR;
    const int32_t nr = (int32_t)(n - r0 < kR ? n - r0 : kR);
    const int32_t pitch = (geo.row_words + 1) | 1;
    const uint32_t q4 = (uint32_t)geo.row_words / 4;
    const uint4 *src = (const uint4 *)(page + r0 * geo.row_words);
    for (uint32_t e = threadIdx.x; e < (uint32_t)nr * q4; e += kR) {
        const uint4 v = src[e];
        const uint32_t r = q4 == 1 ? e : __umulhi(e, q_inv);
        uint32_t *d = rows + r * pitch + (e - r * q4) * 4;
        d[0] = v.x;
        d[1] = v.y;
        d[2] = v.z;
        d[3] = v.w;
    }
    float acc = base;
    const bool mine = (int32_t)threadIdx.x < nr;
    predict_rows<BinStep>(words, chunks, depth, n_chunks, predict_lds, rows + threadIdx.x * pitch, mine, geo.mask,
                          geo.null_sym, &acc);
    if (mine) out[r0 + threadIdx.x] = acc;
}

size_t lds_bytes(int32_t chunk_words, int32_t row_words, int32_t rows)
{
    return ((size_t)chunk_words + (size_t)row_pitch(row_words) * rows) * 4;
}

uint32_t inverse(int32_t d) { return (uint32_t)((((uint64_t)1 << 32) + (uint64_t)d - 1) / (uint64_t)d); }

// One tree in the compact form (tree_words(depth) words); false when a split
// that a walk can reach names no column.
bool compact_tree(const gbt_tree &t, int32_t depth, int32_t w, int32_t n_cols, uint32_t *out)
{
    const int32_t inner = (1 << depth) - 1;
    float *leaf = (float *)(out + 2 * inner);
    // done[i]: i is a leaf or lies below one, whose value is value[i] (the
    // bottom places of the full tree are filled from it); set by the parent
    uint8_t done[(2 << kMaxDepth) - 1];
    float value[(2 << kMaxDepth) - 1];
    done[0] = 0;
    auto settle = [&](int32_t i) {  // a node of the tree: a split, unless it is a leaf or has no children in the table
        const gbt_node &nd = t.nodes[i];
        if (!(nd.flags & GBT_NODE_LEAF) && 2 * (int64_t)i + 2 < t.n_nodes) return;
        done[i] = 1;
        value[i] = nd.leaf_value;
    };
    for (int32_t i = 0; i < inner; ++i) {
        if (!done[i]) settle(i);
        done[2 * i + 1] = done[2 * i + 2] = done[i];
        if (done[i]) {
            value[2 * i + 1] = value[2 * i + 2] = value[i];
            out[2 * i] = out[2 * i + 1] = 0u;
            continue;
        }
        const gbt_node &nd = t.nodes[i];
        const uint32_t def = (nd.flags & GBT_NODE_DEFAULT_LEFT) ? 1u : 0u;
        if (nd.feature < 0 || nd.feature >= n_cols) return false;
        if (w) {
            out[2 * i] = (uint32_t)nd.feature * (uint32_t)w;
            out[2 * i + 1] = 2u * (uint32_t)std::min(std::max(nd.split_bin, 0), 1 << 30) + def;
        } else {
            out[2 * i] = (uint32_t)nd.feature | (def << 31);
            memcpy(&out[2 * i + 1], &nd.threshold, 4);
        }
    }
    for (int32_t i = inner; i < 2 * inner + 1; ++i) leaf[i - inner] = done[i] ? value[i] : t.nodes[i].leaf_value;
    return true;
}

}  // namespace

// Staging a row costs its words whatever the trees read of them, and grows
// with their square, as wider rows leave fewer waves on a CU to hide it; a
// step saves about the same whatever the row.  So the walk in LDS pays from
// steps (of all trees) proportional to the square of the row's loads.  us per
// call, LDS and global, 1 M raw rows: 40 columns 101 / 121 at 6 steps, 50
// columns 118 / 73 at 3 and 118 / 125 at 6, 64 columns 182 / 127 at 6 and 208 /
// 234 at 12 (256 rows a block); 90 columns 467 / 234 at 12 and 560 / 550 at
// 30, 120 columns 871 / 560 at 30 and 916 / 1021 at 60, 300 columns 7928 /
// 3079 at 180 and 9621 / 10053 at 600, 480 columns 11424 / 75 at 3 (64 rows a
// block); 640,000 of 53 columns 119 / 110 at 8.  30,000 rows: 120 columns
// 39 / 33 at 12 and 44 / 52 at 30, 200 columns 78 / 81 at 60, 480 columns 331 /
// 240 at 180 and 465 / 740 at 600; few steps in global memory end as soon
// (26 / 26 at 28 columns and 6 steps; 195 rows of 53 columns 36 / 32 at 12;
// 1.4 M rows of 13 columns 46 / 43 at 2).
// Binned rows take 16-byte loads: 1 M rows of 76 words 114 / 125 at 6 steps, of
// 120 words 281 / 235 at 12 and 301 / 554 at 30.
int32_t lds_predict_rows(const gbt_tree *trees, int32_t n_trees, int64_t n_rows, int32_t row_words, bool binned)
{
    int32_t chunk = kChunkWords;
    int64_t words = 0, steps = 0;
    for (int32_t t = 0; t < n_trees; ++t) {
        if (!trees[t].nodes || trees[t].n_nodes <= 0) return 0;
        const int32_t d = tree_depth(trees[t]);
        if (d > kMaxDepth) return 0;
        chunk = std::max(chunk, tree_words(d));
        words += tree_words(d);
        steps += d;
    }
    if (n_trees == 0 || words > INT32_MAX / 8) return 0;
    const bool few = n_rows <= kFewRows;
    const int32_t rows = !few && lds_bytes(chunk, row_words, 256) <= kLdsRows256 ? 256
                         : lds_bytes(chunk, row_words, 64) <= kLdsRows64         ? 64
                                                                                 : 0;
    const int64_t k = (few ? 400 : rows == 256 ? 300 : 150) * (binned ? 4 : 1);
    if (k * steps < (int64_t)row_words * row_words) return 0;
    if (steps < (!few ? 4 : binned ? 6 : 8 + row_words / 6)) return 0;
    return rows;
}

gbt_status lds_upload_trees(gbt_ctx *c, const gbt_tree *trees, int32_t n_trees, int32_t w, int32_t n_cols,
                            LdsTrees *out, bool *ok)
{
    std::vector<int4> chunks;
    std::vector<int32_t> depth(n_trees);
    int32_t words = 0, most = 0;
    for (int32_t t = 0; t < n_trees; ++t) {
        depth[t] = tree_depth(trees[t]);
        const int32_t n = tree_words(depth[t]);
        if (chunks.empty() || chunks.back().y + n > kChunkWords) chunks.push_back(make_int4(words, 0, t, t));
        chunks.back().y += n;
        chunks.back().w = t + 1;
        words += n;
        most = std::max(most, chunks.back().y);
    }
    const size_t o_chunks = (size_t)words * 4, o_depth = o_chunks + chunks.size() * sizeof(int4);
    const size_t bytes = o_depth + (size_t)n_trees * 4;
    // Pinned memory needs no staging (1000 rows, 10 trees of depth 6: 41 us
    // against 44; 1 M rows, 100 trees of depth 8: 622 against 634), but its
    // allocation takes 50 to 200 us, which that many calls save: until then a
    // context uses it only where it is there already.
    void *host, *dev;
    char *buf;
    if (bytes <= kPinnedTrees && (c->predictions >= kPinnedAfter || c->hio_bytes >= bytes)) {
        GBT_TRY(host_io(c, bytes, &host, &dev));
    } else {
        out->host.resize(bytes);
        host = out->host.data();
    }
    c->predictions = std::min(c->predictions + 1, kPinnedAfter);
    char *h = (char *)host;
    int32_t at = 0;
    *ok = false;
    for (int32_t t = 0; t < n_trees; ++t) {
        if (!compact_tree(trees[t], depth[t], w, n_cols, (uint32_t *)h + at)) return GBT_OK;
        at += tree_words(depth[t]);
    }
    *ok = true;
    memcpy(h + o_chunks, chunks.data(), chunks.size() * sizeof(int4));
    memcpy(h + o_depth, depth.data(), (size_t)n_trees * 4);
    GBT_TRY(scratch_t(c, kScrTrees, bytes, &buf));
    GBT_HIP(hipMemcpyAsync(buf, h, bytes, hipMemcpyHostToDevice, c->stream));
    out->words = (const uint32_t *)buf;
    out->chunks = (const int4 *)(buf + o_chunks);
    out->depth = (const int32_t *)(buf + o_depth);
    out->n_chunks = (int32_t)chunks.size();
    out->chunk_words = most;
    return GBT_OK;
}

gbt_status lds_predict_raw(gbt_ctx *c, const LdsTrees &t, const float *X, int64_t n, int32_t m, int64_t ld, float base,
                           int32_t block_rows, float *out)
{
    const unsigned grid = (unsigned)((n + block_rows - 1) / block_rows);
    const size_t lds = lds_bytes(t.chunk_words, m, block_rows);
    if (block_rows == 256)
        k_predict_raw_lds<256><<<grid, 256, lds, c->stream>>>(X, n, m, ld, inverse(m), t.words, t.chunks, t.depth,
                                                              t.n_chunks, t.chunk_words, base, out);
    else
        k_predict_raw_lds<64><<<grid, 64, lds, c->stream>>>(X, n, m, ld, inverse(m), t.words, t.chunks, t.depth,
                                                            t.n_chunks, t.chunk_words, base, out);
    GBT_LAUNCHED();
    return GBT_OK;
}

gbt_status lds_predict_binned(gbt_ctx *c, const LdsTrees &t, const uint32_t *words, int64_t n, const Geo &geo,
                              float base, int32_t block_rows, float *out)
{
    const unsigned grid = (unsigned)((n + block_rows - 1) / block_rows);
    const size_t lds = lds_bytes(t.chunk_words, geo.row_words, block_rows);
    const uint32_t inv = inverse(geo.row_words / 4);
    if (block_rows == 256)
        k_predict_bin_lds<256><<<grid, 256, lds, c->stream>>>(words, n, geo, inv, t.words, t.chunks, t.depth,
                                                              t.n_chunks, t.chunk_words, base, out);
    else
        k_predict_bin_lds<64><<<grid, 64, lds, c->stream>>>(words, n, geo, inv, t.words, t.chunks, t.depth, t.n_chunks,
                                                            t.chunk_words, base, out);
    GBT_LAUNCHED();
    return GBT_OK;
}

}  // namespace gbt
