// cuts.hip -- exact order statistics of every feature's sketch keys (Sec.
// 3.1, Alg. 2): the values at the ranks ceil(kN/B) - 1 and the largest value.
//
// A segment of up to kSmall keys is sorted by one block in LDS and its ranks
// are read off (k_cut_small).  A longer one is cut into buckets between up
// to 4095 split points taken from a sorted sample of it (k_cut_split), so
// that the buckets hold nearly equal shares whatever the distribution; one
// pass counts the keys per bucket (k_cut_count), which names the bucket of
// every rank (k_cut_plan); a second pass gathers the keys of those buckets
// only (k_cut_gather, about B/4096 of the keys for B bins), and each
// gathered bucket is sorted in LDS for its ranks (k_cut_pick).  The sample
// only decides how even the buckets are: counting is exact, so the results
// do not depend on it.  A value that fills more than one split interval gets
// a bucket of its own, which needs no gathering.
//
// Two passes over the keys instead of a bisection's nine, and no host work
// between them but one read of the gathered size: 500 M keys (50 features x
// 10 M rows, 256 bins) take 2.3 ms against 19.8 ms of bisection passes and
// 8 ms of host sorting between them.
#include "cuts_impl.h"
#include "wave_impl.h"

#include <algorithm>
#include <cstring>

namespace gbt {

namespace {

constexpr uint32_t kNanKey = 0xffffffffu;
constexpr uint32_t kMaxKey = 0xff7fffffu;  // key of the largest finite float
constexpr int kItems = 16;                 // keys per thread in an LDS sort
constexpr int kSmallThreads = 256;         // sorts 4096 keys
constexpr int kBigThreads = 1024;          // sorts 16384 keys
constexpr int kSmall = kBigThreads * kItems;
constexpr int kSample = kBigThreads * kItems;
constexpr int kBuckets = 4096;
constexpr int kCells = 4096;               // cells of the value-linear index over the split points
constexpr int kCountThreads = 512;
constexpr int kPickThreads = 256;          // sorts 1024 or 4096 keys
constexpr int64_t kChunkMin = 1 << 16;     // keys per counting block, at least
constexpr int kChunks = 1024;              // counting blocks, about (every block loads and stores 40 KB of tables)

__device__ inline float key_value(uint32_t k)
{
    return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}

__host__ __device__ inline int64_t cut_rank(int64_t k, int64_t N, int64_t B)
{
    return k < B ? (k * N + B - 1) / B - 1 : N - 1;
}

// LDS place of key i when a thread owns kI keys: one word of padding per
// thread, so that the threads' j-th keys lie in different banks.
template <int kI = kItems>
__device__ inline int pad_idx(int i)
{
    return i + i / kI;
}

// Sorts kT * kI keys, thread t's at positions kI t .. kI t + kI - 1 of sk
// (padded by pad_idx<kI>), in LDS: stable splits by two bits at a time, low
// to high, with the four digit counts in the 16-bit halves of two 32-bit
// scans.  Digits in which no two keys of the block differ are skipped.  The
// fields are 32 bits wide on purpose: with 64-bit ones the compiler put a
// 64-bit vector shift's amount into the last register of the allocation
// (v79 of 80), and gfx950 shifts such a one by another wave's value once two
// blocks share a CU (the build refuses a library that holds one).
template <int kT, int kI = kItems>
__device__ inline void block_sort(uint32_t *sk, uint2 *wsum)
{
    static_assert(kT * kI <= 32768, "16-bit positions");
    constexpr int kWaves = kT / 64;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, base = threadIdx.x * kI;
    __shared__ uint32_t s_or, s_and;
    if (threadIdx.x == 0) {
        s_or = 0u;
        s_and = 0xffffffffu;
    }
    __syncthreads();
    uint32_t k[kI], vo = 0u, va = 0xffffffffu;
#pragma unroll
    for (int j = 0; j < kI; ++j) {
        k[j] = sk[pad_idx<kI>(base + j)];
        // padding and missing keys order last in any digit: every bit is set
        if (k[j] != kNanKey) {
            vo |= k[j];
            va &= k[j];
        }
    }
    vo = wave_fold(vo, [](uint32_t a, uint32_t b) { return a | b; });
    va = wave_fold(va, [](uint32_t a, uint32_t b) { return a & b; });
    if (lane == 0) {
        atomicOr(&s_or, vo);
        atomicAnd(&s_and, va);
    }
    __syncthreads();
    // the bits in which the present keys differ, and the nine top bits, which
    // are all set in missing keys only, so that those order last
    const uint32_t vary = (s_or & ~s_and) | 0xff800000u;
    for (int sh = 0; sh < 32; sh += 2) {
        if (!((vary >> sh) & 3u)) continue;
        // digits 0, 1 in the halves of lo, digits 2, 3 in those of hi
        uint32_t lo = 0, hi = 0;
#pragma unroll
        for (int j = 0; j < kI; ++j) {
            const uint32_t d = (k[j] >> sh) & 3u, one = 1u << (16 * (d & 1u));
            lo += d < 2u ? one : 0u;
            hi += d < 2u ? 0u : one;
        }
        const uint32_t xl = wave_incl_sum(lo), xh = wave_incl_sum(hi);
        if (lane == 63) wsum[wid] = make_uint2(xl, xh);
        __syncthreads();  // also: every thread has read its keys
        uint32_t tl = 0, th = 0;
        lo = xl - lo;
        hi = xh - hi;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            const uint2 v = wsum[w];
            if (w < wid) {
                lo += v.x;
                hi += v.y;
            }
            tl += v.x;
            th += v.y;
        }
        // digit d starts after all keys of lower digits
        const uint32_t low = (tl & 0xffffu) + (tl >> 16);
        lo += tl << 16;
        hi += low * 0x10001u + (th << 16);
#pragma unroll
        for (int j = 0; j < kI; ++j) {
            const uint32_t d = (k[j] >> sh) & 3u, f = 16 * (d & 1u);
            sk[pad_idx<kI>((int)(((d < 2u ? lo : hi) >> f) & 0xffffu))] = k[j];
            lo += d < 2u ? 1u << f : 0u;
            hi += d < 2u ? 0u : 1u << f;
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kI; ++j) k[j] = sk[pad_idx<kI>(base + j)];
    }
    __syncthreads();
}

// Keys of a sorted, padded LDS array that are not missing.
__device__ inline int32_t present_keys(const uint32_t *sk, int32_t n)
{
    int32_t lo = 0, hi = n;
    while (lo < hi) {
        const int32_t mid = (lo + hi) >> 1;
        if (sk[pad_idx(mid)] < kNanKey)
            lo = mid + 1;
        else
            hi = mid;
    }
    return lo;
}

struct CutSeg {
    int64_t begin, len;
    int32_t feat;
    int32_t blk0, blk1;  // its counting blocks
    int32_t pad0;
};

struct CutChunk {
    int64_t begin, end;
    int32_t seg;
    int32_t pad0;
};

// A gathered bucket: cnt keys from off on, and the ranks [r0, r1] it holds.
struct CutPick {
    uint32_t off, cnt;
    int32_t r0, r1;
};

template <int kT>
__global__ void __launch_bounds__(kT)
    k_cut_small(const uint32_t *__restrict__ keys, const CutSeg *__restrict__ segs, int32_t B,
                uint32_t *__restrict__ vals, int64_t *__restrict__ N_out)
{
    __shared__ uint32_t sk[kT * kItems + kT];
    __shared__ uint2 wsum[kT / 64];
    const CutSeg s = segs[blockIdx.x];
    for (int i = threadIdx.x; i < kT * kItems; i += kT) sk[pad_idx(i)] = i < s.len ? keys[s.begin + i] : kNanKey;
    __syncthreads();
    block_sort<kT>(sk, wsum);
    const int64_t N = present_keys(sk, (int32_t)s.len);
    if (threadIdx.x == 0) N_out[s.feat] = N;
    if (N == 0) return;
    for (int32_t k = 1 + threadIdx.x; k <= B; k += kT)
        vals[(int64_t)s.feat * B + k - 1] = sk[pad_idx((int)cut_rank(k, N, B))];
}

// ---- long segments ---------------------------------------------------------
// Tables of one long segment: nb split points b_0 < .. < b_{nb-1} (bucket t
// holds the keys in (b_{t-1}, b_t], bucket nb those above), and an index
// over them by value: cell(x) = the x's place on a linear scale of kCells
// cells over the sample's range (monotone in x, so a key of cell c has its
// split point within [tab[c], tab[c + 1]]).  `steps` halvings settle the
// widest cell.
struct CutTables {
    uint32_t bnd[kBuckets];
    uint16_t tab[kCells + 8];
    int32_t nb, steps;
    float x0, scale;
};
static_assert(sizeof(CutTables) % 16 == 0, "tables are copied in 16-byte pieces");

__device__ inline int32_t cell_of(uint32_t key, float x0, float scale)
{
    // fmax drops a NaN (an infinite difference times a zero scale)
    return (int32_t)fminf(fmaxf((key_value(key) - x0) * scale, 0.0f), (float)(kCells - 1));
}

// A 32-bit integer hash: the constants and shifts are those of Chris Wellons'
// lowbias32, found by his hash prospector and published with it.
__device__ inline uint32_t mix32(uint32_t h)
{
    h ^= h >> 16;
    h *= 0x7feb352du;
    h ^= h >> 15;
    h *= 0x846ca68bu;
    return h ^ (h >> 16);
}

// Split points from a sorted sample, one key from each of kSample equal
// strata at a scrambled place in it (data with a period cannot hide from it).
__global__ void __launch_bounds__(kBigThreads)
    k_cut_split(const uint32_t *__restrict__ keys, const CutSeg *__restrict__ segs, CutTables *__restrict__ tables)
{
    __shared__ uint32_t sk[kSample + kBigThreads];
    __shared__ uint2 wsum[kBigThreads / 64];
    __shared__ int32_t isum[kBigThreads / 64];
    __shared__ int32_t s_wide;
    const CutSeg s = segs[blockIdx.x];
    CutTables &T = tables[blockIdx.x];
    for (int i = threadIdx.x; i < kSample; i += kBigThreads) {
        const int64_t a = (int64_t)i * s.len / kSample, b = (int64_t)(i + 1) * s.len / kSample;
        const int64_t at = a + (int64_t)(mix32((uint32_t)i * 0x9e3779b9u + (uint32_t)s.feat) % (uint32_t)max(b - a, (int64_t)1));
        sk[pad_idx(i)] = keys[s.begin + at];
    }
    if (threadIdx.x == 0) s_wide = 0;
    __syncthreads();
    block_sort<kBigThreads>(sk, wsum);
    const int32_t Ns = present_keys(sk, kSample);
    // q_t = the sample's t-th 4096-quantile.  A quantile met twice or more in
    // a row is a heavy value: the key before it becomes a split point too.
    auto q = [&](int32_t t) -> uint32_t { return sk[pad_idx((int)((int64_t)t * Ns / kBuckets))]; };
    constexpr int kPer = kBuckets / kBigThreads;
    uint32_t out[2 * kPer];
    int32_t n = 0;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const int32_t t = (int32_t)threadIdx.x * kPer + j;
        uint32_t a = 0, b = 0;
        bool two = false, one = false;
        if (t >= 1 && Ns > 0) {
            const uint32_t v = q(t), p = t > 1 ? q(t - 1) : 0u;
            one = t == 1 || v != p;
            two = one && t + 1 < kBuckets && q(t + 1) == v && v > p + 1u;
            a = v - 1u;
            b = v;
        }
        out[2 * j] = two ? a : kNanKey;
        out[2 * j + 1] = one ? b : kNanKey;
        n += (two ? 1 : 0) + (one ? 1 : 0);
    }
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int32_t x = wave_incl_sum(n);
    if (lane == 63) isum[wid] = x;
    __syncthreads();  // the sample is read
    int32_t at = x - n, nb = 0;
    for (int w = 0; w < kBigThreads / 64; ++w) {
        if (w < wid) at += isum[w];
        nb += isum[w];
    }
    const float x0 = Ns ? key_value(sk[0]) : 0.0f;
    float scale = 0.0f;
    if (Ns) {
        const float range = key_value(sk[pad_idx(Ns - 1)]) - x0;
        if (range > 0.0f && range < __builtin_inff()) scale = (float)kCells / range;
        if (!(scale < __builtin_inff())) scale = 0.0f;
    }
    __syncthreads();
    // the split points, in LDS from here on, and in the tables
#pragma unroll
    for (int j = 0; j < 2 * kPer; ++j)
        if (out[j] != kNanKey) {
            sk[at] = out[j];
            T.bnd[at] = out[j];
            ++at;
        }
    for (int32_t t = nb + (int32_t)threadIdx.x; t < kBuckets; t += kBigThreads) T.bnd[t] = kNanKey;
    __syncthreads();
    // tab[c] = split points in cells below c
    uint32_t *cnt = sk + kBuckets;
    for (int32_t c = threadIdx.x; c < kCells; c += kBigThreads) cnt[c] = 0u;
    __syncthreads();
    for (int32_t t = threadIdx.x; t < nb; t += kBigThreads) atomicAdd(&cnt[cell_of(sk[t], x0, scale)], 1u);
    __syncthreads();
    constexpr int kCellPer = kCells / kBigThreads;
    int32_t sum = 0, wide = 0;
#pragma unroll
    for (int j = 0; j < kCellPer; ++j) {
        const int32_t v = (int32_t)cnt[threadIdx.x * kCellPer + j];
        sum += v;
        wide = max(wide, v);
    }
    atomicMax(&s_wide, wide);
    const int32_t y = wave_incl_sum(sum);
    if (lane == 63) isum[wid] = y;
    __syncthreads();
    int32_t o = y - sum;
    for (int w = 0; w < wid; ++w) o += isum[w];
#pragma unroll
    for (int j = 0; j < kCellPer; ++j) {
        T.tab[threadIdx.x * kCellPer + j] = (uint16_t)o;
        o += (int32_t)cnt[threadIdx.x * kCellPer + j];
    }
    if (threadIdx.x == 0) {
        for (int c = kCells; c < kCells + 8; ++c) T.tab[c] = (uint16_t)nb;
        int32_t steps = 0;
        while ((1 << steps) < s_wide + 1) ++steps;
        T.nb = nb;
        T.steps = steps;
        T.x0 = x0;
        T.scale = scale;
    }
}

// The segment's tables in LDS.
struct CutLds {
    CutTables T;
    uint32_t cnt[kBuckets];
};

__device__ inline void load_tables(const CutTables *__restrict__ src, CutTables *dst)
{
    const uint4 *a = (const uint4 *)src;
    uint4 *b = (uint4 *)dst;
    for (int i = threadIdx.x; i < (int)(sizeof(CutTables) / 16); i += kCountThreads) b[i] = a[i];
}

// Buckets of kU keys at once (independent searches, so that their LDS reads
// overlap).
template <int kU>
__device__ inline void find_buckets(const CutTables &T, int32_t steps, float x0, float scale, const uint32_t (&k)[kU],
                                    int32_t (&lo)[kU])
{
    int32_t hi[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
        const int32_t c = cell_of(k[u], x0, scale);
        lo[u] = T.tab[c];
        hi[u] = T.tab[c + 1];
    }
    for (int s = 0; s < steps; ++s) {
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int32_t mid = (lo[u] + hi[u]) >> 1;
            // mid <= nb <= kBuckets - 1; entries from nb on are the NaN key
            const bool below = T.bnd[mid] < k[u], open = lo[u] < hi[u];
            lo[u] = open && below ? mid + 1 : lo[u];
            hi[u] = open && !below ? mid : hi[u];
        }
    }
}

constexpr int kUnroll = 8;

// Counts of one chunk's keys per bucket: part[blockIdx.x][t].  Bound by the
// key reads and the LDS (two index reads, `steps` halvings and one atomic
// per key).
__global__ void __launch_bounds__(kCountThreads)
    k_cut_count(const uint32_t *__restrict__ keys, const CutChunk *__restrict__ chunks,
                const CutTables *__restrict__ tables, uint32_t *__restrict__ part)
{
    __shared__ __align__(16) CutLds L;
    const CutChunk ch = chunks[blockIdx.x];
    load_tables(tables + ch.seg, &L.T);
    for (int t = threadIdx.x; t < kBuckets; t += kCountThreads) L.cnt[t] = 0u;
    __syncthreads();
    const int32_t steps = L.T.steps;
    const float x0 = L.T.x0, scale = L.T.scale;
    for (int64_t i0 = ch.begin; i0 < ch.end; i0 += kCountThreads * kUnroll) {
        uint32_t k[kUnroll];
        int32_t b[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const int64_t i = i0 + u * kCountThreads + threadIdx.x;
            k[u] = i < ch.end ? keys[i] : kNanKey;
        }
        find_buckets(L.T, steps, x0, scale, k, b);
#pragma unroll
        for (int u = 0; u < kUnroll; ++u)
            if (k[u] != kNanKey) atomicAdd(&L.cnt[b[u]], 1u);
    }
    __syncthreads();
    for (int t = threadIdx.x; t < kBuckets; t += kCountThreads) part[(int64_t)blockIdx.x * kBuckets + t] = L.cnt[t];
}

// One block per long segment: the chunks' counts become each chunk's first
// place in its buckets, the ranks find their buckets; a rank in a bucket of
// one value is answered, the other buckets that hold a rank are laid out
// one after the other for gathering (place[t], kNanKey for the rest).
__global__ void __launch_bounds__(kBigThreads)
    k_cut_plan(const CutSeg *__restrict__ segs, const CutTables *__restrict__ tables, uint32_t *__restrict__ part,
               int32_t B, uint32_t *__restrict__ vals, int64_t *__restrict__ N_out, uint32_t *__restrict__ place,
               CutPick *__restrict__ picks, int32_t max_picks, uint32_t *__restrict__ rank_res,
               int64_t *__restrict__ gather_n)
{
    __shared__ uint32_t ex[kBuckets];    // keys below the bucket
    __shared__ int32_t rmin[kBuckets], rmax[kBuckets];
    __shared__ uint32_t wsum[kBigThreads / 64], wsum2[kBigThreads / 64];
    const CutSeg s = segs[blockIdx.x];
    const CutTables &T = tables[blockIdx.x];
    constexpr int kPer = kBuckets / kBigThreads;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int32_t t0 = (int32_t)threadIdx.x * kPer;
    uint32_t cnt[kPer] = {};
    for (int32_t b = s.blk0; b < s.blk1; ++b) {
        uint4 *p = (uint4 *)(part + (int64_t)b * kBuckets + t0);
        static_assert(kPer == 4, "one 16-byte piece per thread");
        const uint4 v = *p;
        *p = make_uint4(cnt[0], cnt[1], cnt[2], cnt[3]);
        cnt[0] += v.x;
        cnt[1] += v.y;
        cnt[2] += v.z;
        cnt[3] += v.w;
    }
    uint32_t sum = cnt[0] + cnt[1] + cnt[2] + cnt[3];
    const uint32_t x = wave_incl_sum(sum);
    if (lane == 63) wsum[wid] = x;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        rmin[t0 + j] = INT32_MAX;
        rmax[t0 + j] = -1;
    }
    __syncthreads();
    uint32_t o = x - sum, N32 = 0;
    for (int w = 0; w < kBigThreads / 64; ++w) {
        if (w < wid) o += wsum[w];
        N32 += wsum[w];
    }
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        ex[t0 + j] = o;
        o += cnt[j];
    }
    __syncthreads();
    const int64_t N = N32;
    if (threadIdx.x == 0) N_out[s.feat] = N;
    const int32_t nb = T.nb;
    auto single = [&](int32_t t) {
        const int64_t below = t ? (int64_t)T.bnd[t - 1] : -1;
        return (t < nb ? (int64_t)T.bnd[t] : (int64_t)kMaxKey) - below == 1;
    };
    if (N > 0)
        for (int32_t k = 1 + threadIdx.x; k <= B; k += kBigThreads) {
            const uint32_t r = (uint32_t)cut_rank(k, N, B);
            int32_t lo = 0, hi = kBuckets;  // the last bucket with ex <= r holds rank r
            while (hi - lo > 1) {
                const int32_t mid = (lo + hi) >> 1;
                if (ex[mid] <= r)
                    lo = mid;
                else
                    hi = mid;
            }
            if (single(lo)) {
                vals[(int64_t)s.feat * B + k - 1] = lo < nb ? T.bnd[lo] : kMaxKey;
            } else {
                rank_res[(int64_t)s.feat * B + k - 1] = r - ex[lo];
                atomicMin(&rmin[lo], k - 1);
                atomicMax(&rmax[lo], k - 1);
            }
        }
    __syncthreads();
    uint32_t need = 0, items = 0;
#pragma unroll
    for (int j = 0; j < kPer; ++j)
        if (rmax[t0 + j] >= 0) {
            need += cnt[j];
            ++items;
        }
    const uint32_t y = wave_incl_sum(need), z = wave_incl_sum(items);
    if (lane == 63) {
        wsum[wid] = y;
        wsum2[wid] = z;
    }
    __syncthreads();
    uint32_t g = y - need, it = z - items, total = 0, n_items = 0;
    for (int w = 0; w < kBigThreads / 64; ++w) {
        if (w < wid) {
            g += wsum[w];
            it += wsum2[w];
        }
        total += wsum[w];
        n_items += wsum2[w];
    }
    CutPick *pk = picks + (int64_t)blockIdx.x * max_picks;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const bool in = rmax[t0 + j] >= 0;
        place[(int64_t)blockIdx.x * kBuckets + t0 + j] = in ? g : kNanKey;
        if (in) {
            pk[it] = {g, cnt[j], rmin[t0 + j], rmax[t0 + j]};
            g += cnt[j];
            ++it;
        }
    }
    if (threadIdx.x == 0) {
        gather_n[2 * blockIdx.x] = total;
        gather_n[2 * blockIdx.x + 1] = n_items;
    }
}

// Orders a wave's LDS writes before its later reads of other lanes' words.
__device__ inline void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The keys of the buckets to be gathered, bucket by bucket (any order
// within one): the chunk's first place in a bucket is known, so only LDS
// cursors are needed.  Most cells of the index hold no gathered bucket (256
// bins: 6 % of the keys are gathered), so a bit per cell drops most keys
// after one LDS read; a wave lines the others up in LDS and searches them 64
// at a time.  500 M keys of 50 features 863 us against 1026 with every key
// searched, 28 M of 28 features 59 against 67; 40 M of 2000 features (short
// chunks, which the bits' set-up weighs on) 101 against 94.
__global__ void __launch_bounds__(kCountThreads)
    k_cut_gather(const uint32_t *__restrict__ keys, const CutChunk *__restrict__ chunks,
                 const CutTables *__restrict__ tables, const uint32_t *__restrict__ part,
                 const uint32_t *__restrict__ place, const int64_t *__restrict__ base, uint32_t *__restrict__ out)
{
    __shared__ __align__(16) CutLds L;
    __shared__ uint32_t hit[kCells / 32];
    __shared__ uint32_t line[kCountThreads * 2];
    const CutChunk ch = chunks[blockIdx.x];
    load_tables(tables + ch.seg, &L.T);
    for (int t = threadIdx.x; t < kBuckets; t += kCountThreads) {
        const uint32_t p = place[(int64_t)ch.seg * kBuckets + t];
        L.cnt[t] = p == kNanKey ? kNanKey : p + part[(int64_t)blockIdx.x * kBuckets + t];
    }
    if (threadIdx.x < kCells / 32) hit[threadIdx.x] = 0u;
    __syncthreads();
    // cell c's keys lie in buckets tab[c] .. tab[c + 1]
    for (int c = threadIdx.x; c < kCells; c += kCountThreads) {
        bool any = false;
        for (int t = L.T.tab[c]; t <= L.T.tab[c + 1] && !any; ++t) any = L.cnt[t] != kNanKey;
        if (any) atomicOr(&hit[c >> 5], 1u << (c & 31));
    }
    __syncthreads();
    uint32_t *dst = out + base[ch.seg];
    const int32_t steps = L.T.steps;
    const float x0 = L.T.x0, scale = L.T.scale;
    const int lane = threadIdx.x & 63;
    uint32_t *mine = line + (threadIdx.x >> 6) * 128;  // the wave's, at most 63 kept and 64 new
    int32_t n = 0;  // keys in line (the same in every lane)
    auto search = [&](uint32_t key) {
        const uint32_t v[1] = {key};
        int32_t b[1];
        find_buckets(L.T, steps, x0, scale, v, b);
        if (key != kNanKey && L.cnt[b[0]] != kNanKey) dst[atomicAdd(&L.cnt[b[0]], 1u)] = key;
    };
    for (int64_t i0 = ch.begin; i0 < ch.end; i0 += kCountThreads * kUnroll) {
        uint32_t k[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const int64_t i = i0 + u * kCountThreads + threadIdx.x;
            k[u] = i < ch.end ? keys[i] : kNanKey;
        }
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const int32_t c = cell_of(k[u], x0, scale);
            const bool take = k[u] != kNanKey && ((hit[c >> 5] >> (c & 31)) & 1u);
            const uint64_t m = __ballot(take);
            if (take) mine[n + lanes_below(m)] = k[u];
            n += __popcll(m);
            if (n >= 64) {
                wave_lds_fence();
                const uint32_t key = mine[lane], rest = mine[64 + lane];
                wave_lds_fence();
                n -= 64;
                if (lane < n) mine[lane] = rest;
                search(key);
            }
        }
    }
    wave_lds_fence();
    search(lane < n ? mine[lane] : kNanKey);
}

// The ranks pk.r0 .. pk.r1 of a bucket of up to kPickThreads * kI keys.
template <int kI>
__device__ inline void pick_sorted(const uint32_t *a, const CutPick &pk, const uint32_t *__restrict__ rank_res,
                                   uint32_t *__restrict__ vals, uint32_t *sk, uint2 *wsum)
{
    constexpr uint32_t kCap = kPickThreads * kI;
    for (uint32_t i = threadIdx.x; i < kCap; i += kPickThreads) sk[pad_idx<kI>(i)] = i < pk.cnt ? a[i] : kNanKey;
    __syncthreads();
    block_sort<kPickThreads, kI>(sk, wsum);
    for (int32_t r = pk.r0 + (int32_t)threadIdx.x; r <= pk.r1; r += kPickThreads)
        vals[r] = sk[pad_idx<kI>((int)rank_res[r])];
}

// Block (i, s): the ranks of segment s's i-th gathered bucket.  A bucket of
// up to 4096 keys is sorted in LDS (up to 1024 with a quarter of the keys
// per thread: the passes' barriers, not their keys, set a block's time, and
// buckets of 250 keys took 390 us per 7,000 in a 512-thread block of 16 keys
// a thread); a larger one is searched rank by rank, eight bits at a time.
__global__ void __launch_bounds__(kPickThreads)
    k_cut_pick(const uint32_t *__restrict__ gathered, const int64_t *__restrict__ base,
               const CutSeg *__restrict__ segs, const CutPick *__restrict__ picks, int32_t max_picks,
               const int64_t *__restrict__ gather_n, const uint32_t *__restrict__ rank_res, int32_t B,
               uint32_t *__restrict__ vals)
{
    __shared__ uint32_t sk[kPickThreads * kItems + kPickThreads];
    __shared__ uint2 wsum[kPickThreads / 64];
    __shared__ uint32_t s_digit, s_below;
    if ((int64_t)blockIdx.x >= gather_n[2 * blockIdx.y + 1]) return;
    const CutPick pk = picks[(int64_t)blockIdx.y * max_picks + blockIdx.x];
    const uint32_t *a = gathered + base[blockIdx.y] + pk.off;
    const int64_t at = (int64_t)segs[blockIdx.y].feat * B;
    if (pk.cnt <= kPickThreads * 4) {
        pick_sorted<4>(a, pk, rank_res + at, vals + at, sk, wsum);
        return;
    }
    if (pk.cnt <= kPickThreads * kItems) {
        pick_sorted<kItems>(a, pk, rank_res + at, vals + at, sk, wsum);
        return;
    }
    for (int32_t r = pk.r0; r <= pk.r1; ++r) {
        uint32_t want = rank_res[at + r], prefix = 0;
        for (int sh = 24; sh >= 0; sh -= 8) {
            for (int d = threadIdx.x; d < 256; d += kPickThreads) sk[d] = 0u;
            __syncthreads();
            const uint32_t mask = sh == 24 ? 0u : 0xffffffffu << (sh + 8);
            for (uint32_t i = threadIdx.x; i < pk.cnt; i += kPickThreads) {
                const uint32_t k = a[i];
                if ((k & mask) == prefix) atomicAdd(&sk[(k >> sh) & 255u], 1u);
            }
            __syncthreads();
            if (threadIdx.x < 64) {  // the digit whose keys hold rank `want`: four digits per lane
                const uint32_t *d4 = sk + 4 * threadIdx.x;
                const uint32_t sum = d4[0] + d4[1] + d4[2] + d4[3], incl = wave_incl_sum(sum);
                uint32_t below = incl - sum;
                if (below <= want && want < incl) {
                    uint32_t d = 0;
                    while (below + d4[d] <= want) below += d4[d++];
                    s_digit = 4 * threadIdx.x + d;
                    s_below = below;
                }
            }
            __syncthreads();
            prefix |= s_digit << sh;
            want -= s_below;
            __syncthreads();
        }
        if (threadIdx.x == 0) vals[at + r] = prefix;
    }
}

}  // namespace

gbt_status select_cut_keys(gbt_ctx *c, const uint32_t *keys, const std::vector<int64_t> &seg, int32_t max_bin,
                           std::vector<uint32_t> *vals, std::vector<int64_t> *N)
{
    const int32_t m = (int32_t)seg.size() - 1, B = max_bin;
    // the segments by kind (long ones first), and the long ones' chunks
    std::vector<CutSeg> segs, mid, small;
    int64_t long_keys = 0;
    for (int32_t j = 0; j < m; ++j) {
        const int64_t len = seg[j + 1] - seg[j];
        // keys are counted, ranked and stepped over in 32 unsigned bits
        GBT_CHECK(len >= 0 && len <= (int64_t)UINT32_MAX - kSmall, "feature %d has %lld sketch keys", j, (long long)len);
        const CutSeg s{seg[j], len, j, 0, 0, 0};
        if (len > kSmall) {
            segs.push_back(s);
            long_keys += len;
        } else if (len > kSmallThreads * kItems) {
            mid.push_back(s);
        } else if (len > 0) {
            small.push_back(s);
        }
    }
    const int32_t n_long = (int32_t)segs.size(), n_mid = (int32_t)mid.size(), n_small = (int32_t)small.size();
    std::vector<CutChunk> chunks;
    const int64_t chunk = std::max(kChunkMin, (long_keys + kChunks - 1) / kChunks);
    for (int32_t i = 0; i < n_long; ++i) {
        segs[i].blk0 = (int32_t)chunks.size();
        for (int64_t b = 0; b < segs[i].len; b += chunk)
            chunks.push_back({segs[i].begin + b, segs[i].begin + std::min(segs[i].len, b + chunk), i, 0});
        segs[i].blk1 = (int32_t)chunks.size();
    }
    segs.insert(segs.end(), mid.begin(), mid.end());
    segs.insert(segs.end(), small.begin(), small.end());
    const size_t n_blk = chunks.size();
    const int32_t max_picks = std::min(B, kBuckets);

    // one workspace: results | segments | chunks | tables | counts | places |
    // picks | residual ranks | gathered sizes | gathered bases
    size_t total = 0;
    auto part = [&](size_t bytes) {
        const size_t at = total;
        total += (bytes + 255) / 256 * 256;
        return at;
    };
    const size_t o_vals = part((size_t)m * B * 4), o_N = part((size_t)m * 8);
    const size_t o_segs = part(segs.size() * sizeof(CutSeg)), o_chunks = part(n_blk * sizeof(CutChunk));
    const size_t o_tab = part((size_t)n_long * sizeof(CutTables)), o_part = part(n_blk * kBuckets * 4);
    const size_t o_place = part((size_t)n_long * kBuckets * 4);
    const size_t o_picks = part((size_t)n_long * max_picks * sizeof(CutPick));
    const size_t o_res = part(n_long ? (size_t)m * B * 4 : 0);
    const size_t o_gn = part((size_t)n_long * 16), o_base = part((size_t)n_long * 8);
    char *w = nullptr;
    GBT_TRY(dev_alloc(c, total, (void **)&w));
    uint32_t *gathered = nullptr;
    size_t gathered_bytes = 0;
    std::vector<char> up(o_tab - o_segs);
    std::vector<int64_t> gn((size_t)n_long * 2), base((size_t)n_long);
    auto run = [&]() -> gbt_status {
        memset(up.data(), 0, up.size());
        if (!segs.empty()) memcpy(up.data(), segs.data(), segs.size() * sizeof(CutSeg));
        if (n_blk) memcpy(up.data() + (o_chunks - o_segs), chunks.data(), n_blk * sizeof(CutChunk));
        if (!up.empty()) GBT_HIP(hipMemcpyAsync(w + o_segs, up.data(), up.size(), hipMemcpyHostToDevice, c->stream));
        uint32_t *vals_d = (uint32_t *)(w + o_vals);
        int64_t *N_d = (int64_t *)(w + o_N);
        const CutSeg *segs_d = (const CutSeg *)(w + o_segs);
        const CutChunk *chunks_d = (const CutChunk *)(w + o_chunks);
        CutTables *tab_d = (CutTables *)(w + o_tab);
        uint32_t *part_d = (uint32_t *)(w + o_part), *place_d = (uint32_t *)(w + o_place);
        CutPick *picks_d = (CutPick *)(w + o_picks);
        uint32_t *res_d = (uint32_t *)(w + o_res);
        int64_t *gn_d = (int64_t *)(w + o_gn), *base_d = (int64_t *)(w + o_base);
        if (n_long) {
            k_cut_split<<<n_long, kBigThreads, 0, c->stream>>>(keys, segs_d, tab_d);
            GBT_LAUNCHED();
            k_cut_count<<<(unsigned)n_blk, kCountThreads, 0, c->stream>>>(keys, chunks_d, tab_d, part_d);
            GBT_LAUNCHED();
            k_cut_plan<<<n_long, kBigThreads, 0, c->stream>>>(segs_d, tab_d, part_d, B, vals_d, N_d, place_d, picks_d,
                                                              max_picks, res_d, gn_d);
            GBT_LAUNCHED();
            GBT_HIP(hipMemcpyAsync(gn.data(), gn_d, gn.size() * 8, hipMemcpyDeviceToHost, c->stream));
        }
        if (n_mid) {
            k_cut_small<kBigThreads><<<n_mid, kBigThreads, 0, c->stream>>>(keys, segs_d + n_long, B, vals_d, N_d);
            GBT_LAUNCHED();
        }
        if (n_small) {
            k_cut_small<kSmallThreads><<<n_small, kSmallThreads, 0, c->stream>>>(keys, segs_d + n_long + n_mid, B,
                                                                                 vals_d, N_d);
            GBT_LAUNCHED();
        }
        if (n_long) {
            GBT_HIP(hipStreamSynchronize(c->stream));
            int64_t sum = 0, most = 0;
            for (int32_t i = 0; i < n_long; ++i) {
                base[i] = sum;
                sum += gn[2 * i];
                most = std::max(most, gn[2 * i + 1]);
            }
            if (most > 0) {
                gathered_bytes = (size_t)sum * 4;
                gbt_status s = dev_alloc(c, gathered_bytes, (void **)&gathered);
                if (s != GBT_OK) {
                    gathered_bytes = 0;
                    return s;
                }
                GBT_HIP(hipMemcpyAsync(base_d, base.data(), base.size() * 8, hipMemcpyHostToDevice, c->stream));
                k_cut_gather<<<(unsigned)n_blk, kCountThreads, 0, c->stream>>>(keys, chunks_d, tab_d, part_d, place_d,
                                                                               base_d, gathered);
                GBT_LAUNCHED();
                k_cut_pick<<<dim3((unsigned)most, (unsigned)n_long), kPickThreads, 0, c->stream>>>(
                    gathered, base_d, segs_d, picks_d, max_picks, gn_d, res_d, B, vals_d);
                GBT_LAUNCHED();
            }
        }
        vals->assign((size_t)m * B, 0u);
        N->assign(m, 0);
        GBT_HIP(hipMemcpyAsync(vals->data(), vals_d, (size_t)m * B * 4, hipMemcpyDeviceToHost, c->stream));
        GBT_HIP(hipMemcpyAsync(N->data(), N_d, (size_t)m * 8, hipMemcpyDeviceToHost, c->stream));
        GBT_HIP(hipStreamSynchronize(c->stream));
        for (int32_t j = 0; j < m; ++j)
            if (seg[j + 1] == seg[j]) (*N)[j] = 0;  // no block wrote its count
        return GBT_OK;
    };
    const gbt_status s = run();
    (void)hipStreamSynchronize(c->stream);
    dev_free(c, gathered, gathered_bytes);
    dev_free(c, w, total);
    return s;
}

}  // namespace gbt
