// gfx950 kernels of the SINDI search path (arXiv 2509.08395).
//
//   k_query_prep   validate query rows; beta-mass subvector (Def. 6, Sec. 4.1)
//   k_accumulate1  stream each query term's window list I_{j,w} (Alg. 2,
//                  product + accumulate steps) into an on-chip score tile,
//                  one query per workgroup, the waves taking batches of
//                  chunks from a counter; then either sample per-thread
//                  maxima (threshold pass) or emit every tile score at or
//                  above the query's threshold (k_accumulate1_queue: the same
//                  as one persistent launch fed by a device queue)
//   k_accumulate   the same for batches of 2, 4 or 8 queries sharing lists
//   k_theta        per-query candidate threshold from the sampled maxima
//   k_finalize     exact top-gamma of the emitted candidates (Alg. 2 heap
//                  update): into the rerank pool, or sorted into the coarse
//                  top-k (Alg. 2 alone)
//   k_rerank       exact FP32 rerank of the pool from the unpruned vectors
//                  (Alg. 4), four pool entries per wave
//   k_topk         top-k of the reranked pool (Alg. 4)
//   k_score_*      delta(q, x) of listed pairs (Def. 2) and its gradient
//
// Ranking order: score descending, then document id ascending.  A candidate
// is one 64-bit key: (order-preserving score bits << 32) | (~doc id), so the
// ranking order is plain descending key order and keys are unique.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <algorithm>
#include <map>
#include <mutex>
#include <tuple>
#include <type_traits>
#include <utility>

#include "sindi_internal.h"

namespace sindi {
namespace {

constexpr int kWave = 64;
constexpr int kRerankPerWave = 4;  // pool entries one rerank wave scores at a time
constexpr int kRerankGroups = 4;   // most such groups per wave (one query table per workgroup)
constexpr uint32_t kCandBuf = 256;  // candidates a scoring workgroup holds in LDS
constexpr int kFewHits = 4;        // lanes that place their candidates one by one
constexpr int kRankSort = 256;     // most keys put in order by counting the larger ones
constexpr int kTopkRegs = 8;       // pool keys per thread of a selecting k_topk
constexpr int64_t kRerankFill = 2048;  // rerank workgroups that fill the chip
constexpr int kMaxSeg = kQueryHash / 2 / kWave;  // 64-term segments of the longest query
constexpr int kPrepWaves = 8;      // query rows per prep workgroup, one wave each
constexpr int kPrepRow = 512;      // longest query row a prep wave holds in registers and LDS

__device__ __forceinline__ uint32_t ord_f32(float f)
{
    uint32_t u = __float_as_uint(f);
    if (f == 0.0f) u = 0u;  // -0 ranks as +0
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float unord_f32(uint32_t o)
{
    return __uint_as_float((o & 0x80000000u) ? (o & 0x7FFFFFFFu) : ~o);
}
__device__ __forceinline__ uint64_t make_key(float s, uint32_t doc)
{
    return ((uint64_t)ord_f32(s) << 32) | (uint64_t)(0xFFFFFFFFu - doc);
}
__device__ __forceinline__ uint32_t key_doc(uint64_t k) { return 0xFFFFFFFFu - (uint32_t)k; }
__device__ __forceinline__ float key_score(uint64_t k) { return unord_f32((uint32_t)(k >> 32)); }

// A zero vector materialised where it is used (a plain register move the
// compiler cannot hoist out of the loop and keep live, or spill, at high
// register pressure).
__device__ __forceinline__ int4 fresh_zero4()
{
    int32_t z;
    asm volatile("v_mov_b32 %0, 0" : "=v"(z));
    return make_int4(z, z, z, z);
}

// Wave-uniform copy of a value (scalar register).
__device__ __forceinline__ uint32_t uni(uint32_t x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ int64_t uni64(int64_t x)
{
    return (int64_t)(((uint64_t)uni((uint32_t)((uint64_t)x >> 32)) << 32) | uni((uint32_t)x));
}
__device__ __forceinline__ int64_t readlane64(int64_t x, int l)
{
    return (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(x >> 32), l) << 32) |
                     (uint32_t)__builtin_amdgcn_readlane((int)x, l));
}
// A wave-uniform pointer to global memory, held in scalar registers, and
// loads of 8 or 16 bytes at a 32-bit byte offset from it (the scalar base +
// vector offset form of the global load).
using gbytes = const unsigned char __attribute__((address_space(1))) *;
__device__ __forceinline__ gbytes uni_ptr(const void *p)
{
    const uint64_t a = reinterpret_cast<uint64_t>(p);
    return (gbytes)(((uint64_t)uni((uint32_t)(a >> 32)) << 32) | uni((uint32_t)a));
}
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void load_at(gbytes p, uint32_t off, uint2 &r)
{
    const u32x2 v = *(const u32x2 __attribute__((address_space(1))) *)(p + off);
    r = make_uint2(v.x, v.y);
}
__device__ __forceinline__ void load_at(gbytes p, uint32_t off, uint4 &r)
{
    const u32x4 v = *(const u32x4 __attribute__((address_space(1))) *)(p + off);
    r = make_uint4(v.x, v.y, v.z, v.w);
}

__device__ __forceinline__ uint32_t lanes_below(uint64_t m)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

__device__ __forceinline__ void lds_add(float *p, float v)
{
    __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
// Integer LDS atomics run at many times the rate of float ones on gfx950.
__device__ __forceinline__ void lds_add_i32(int32_t *p, int32_t v)
{
    __hip_atomic_fetch_add(reinterpret_cast<uint32_t *>(p), (uint32_t)v, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Read and clear in one pass: an LDS exchange (8 and 4 cycles of the LDS a wave for 8 and 4 bytes a
// lane) does both in the time that the 16-byte write alone takes.  Scoring pass over 7,000 queries and
// 8.8M documents 46.4 -> 46.0 ms, with alpha 0.2, beta 0.8 17.8 -> 17.4 ms.
__device__ __forceinline__ int32_t lds_take(int32_t *p)
{
    return (int32_t)__hip_atomic_exchange(reinterpret_cast<uint32_t *>(p), 0u, __ATOMIC_RELAXED,
                                          __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ int4 lds_take4(int32_t *p)  // p 16-byte aligned
{
    uint64_t *q = reinterpret_cast<uint64_t *>(p);
    const uint64_t x = __hip_atomic_exchange(q, (uint64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    const uint64_t y = __hip_atomic_exchange(q + 1, (uint64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    return make_int4((int32_t)(uint32_t)x, (int32_t)(x >> 32), (int32_t)(uint32_t)y, (int32_t)(y >> 32));
}

// Exclusive scan of one value per thread over the block; `total` = sum.
template <int NT>
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t *wsum, uint32_t &total)
{
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    uint32_t x = v;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        uint32_t y = __shfl_up(x, d, kWave);
        if (lane >= d) x += y;
    }
    if (lane == kWave - 1) wsum[wave] = x;
    __syncthreads();
    uint32_t off = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < NT / kWave; ++i) {
        uint32_t s = wsum[i];
        off += (i < wave) ? s : 0u;
        tot += s;
    }
    total = tot;
    __syncthreads();
    return off + x - v;
}

// Inclusive prefix sum over the wave in lane order: within each row of 16
// lanes by four shifted adds (DPP row_shr 1, 2, 4, 8; lanes shifted in from
// outside the row read 0), then rows 1 and 3 add the total of the row below, then the upper half
// that of the lower (DPP row_bcast 15 and 31).
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t x)
{
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, false);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xF, 0xF, false);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xF, 0xF, false);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xF, 0xF, false);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xA, 0xF, false);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xC, 0xF, false);
    return x;
}

// LDS of a block_select.
struct SelectLds {
    uint32_t hist[2][256];
    uint64_t differ[16];  // per wave: the bits in which its keys differ from the first key
    uint32_t digit, need, count;
};

// Radix select over the workgroup's keys: each(f) calls f on every key the calling thread owns,
// `any` is one of the keys (the same on every thread), 1 <= r <= number of keys.  Returns a bound
// t: the keys at or above t are the r largest (more only where keys tie at t, which is then the
// r-th largest key itself).  *exact: t is that key.
//
// The digits start at the highest bit in which keys differ (scores share their upper bits) and
// stop once the digits chosen so far hold just the keys still needed, so 64-bit keys take two or
// three passes of 8 bits, not eight, each of two barriers.
template <int NT, typename K, typename Each>
__device__ __forceinline__ K block_select(K any, int64_t r, Each each, SelectLds &L, bool *exact)
{
    static_assert(NT / kWave <= 16 && NT >= 256, "SelectLds");
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    K x = 0;
    each([&](K k) { x |= k ^ any; });
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) x |= __shfl_xor(x, m, kWave);
    if (lane == 0) L.differ[tid / kWave] = (uint64_t)x;
    if (tid < 256) L.hist[0][tid] = 0u;
    __syncthreads();
    uint64_t diff = 0;
#pragma unroll
    for (int i = 0; i < NT / kWave; ++i) diff |= L.differ[i];
    int top = diff ? 64 - __clzll((long long)diff) : 0;  // bits still undecided
    K mask = top >= (int)sizeof(K) * 8 ? (K)0 : (K)(~(K)0 << top);
    K prefix = any & mask;
    uint32_t need = (uint32_t)r;
    bool whole = false;  // the digits so far hold just the keys still needed
    for (int cur = 0; top > 0 && !whole; cur ^= 1) {
        const int shift = max(0, top - 8);
        const uint32_t dmask = (1u << (top - shift)) - 1u;
        if (tid < 256) L.hist[cur ^ 1][tid] = 0u;
        each([&](K k) {
            if ((k & mask) == prefix) atomicAdd(&L.hist[cur][(uint32_t)(k >> shift) & dmask], 1u);
        });
        __syncthreads();
        if (tid < kWave) {
            // digit of the need-th key: lane l holds digits 255 - 4l .. 252 - 4l; a prefix
            // sum over the lanes counts the keys with larger digits
            uint32_t h[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) h[u] = L.hist[cur][255 - 4 * tid - u];
            const uint32_t tot = h[0] + h[1] + h[2] + h[3];
            const uint32_t incl = wave_incl_scan(tot);
            uint32_t acc = incl - tot;
            if (acc < need && incl >= need) {
                int u = 0;
                while (u < 3 && acc + h[u] < need) acc += h[u++];
                L.digit = (uint32_t)(255 - 4 * tid - u);
                L.need = need - acc;
                L.count = h[u];
            }
        }
        __syncthreads();
        prefix |= (K)L.digit << shift;
        mask |= (K)dmask << shift;
        need = L.need;
        whole = L.count == need;
        top = shift;
    }
    if (exact) *exact = top == 0;
    __syncthreads();  // L may be used again
    return prefix;
}

// ------------------------------------------------------------------ queries
// Orders a wave's LDS accesses against each other (one wave's DS operations execute in order;
// this keeps the compiler from moving them).
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// LDS of one prep wave: the row's ranking keys, later its kept entries.
struct PrepRow {
    union {
        uint64_t key[kPrepRow];
        struct {
            int32_t id[kPrepRow];
            float w[kPrepRow];
        };
    };
    float abs[kPrepRow];  // |x| by rank
};

// Entries of a row of n <= 64 J held J per lane (entry 64 j + lane in slot j; id, v; absent and
// zero entries have key 0): bit j of the result is set for the slots Def. 6's prefix keeps.
template <int J>
__device__ __forceinline__ uint32_t beta_mass_keep(const uint64_t (&key)[J], int32_t n, double beta,
                                                   PrepRow &r)
{
    const int lane = threadIdx.x & (kWave - 1);
    int32_t rank[J], nz = 0;
#pragma unroll
    for (int j = 0; j < J; ++j) {
        r.key[j * kWave + lane] = key[j];
        rank[j] = 0;
        nz += (int32_t)__popcll(__ballot(key[j] != 0));
    }
    wave_lds_sync();
    // rank of every entry in pi order: the keys above its own (zero keys are above none)
    for (int32_t f = 0; f < n; f += 8) {  // past n: zero keys
        uint64_t k[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) k[i] = r.key[f + i];
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int j = 0; j < J; ++j) rank[j] += k[i] > key[j] ? 1 : 0;
    }
#pragma unroll
    for (int j = 0; j < J; ++j)
        if (key[j]) r.abs[rank[j]] = __uint_as_float((uint32_t)(key[j] >> 32));
    wave_lds_sync();
    // FP64 prefix sums in rank order, one addition after another; lane l keeps the sums of
    // ranks l, l + 64, ...  The last one is the mass.
    double run = 0.0, pre[J];
#pragma unroll
    for (int j = 0; j < J; ++j) {
        pre[j] = 0.0;
        const int32_t m = min(kWave, nz - j * kWave);
        const int av = __float_as_int(r.abs[j * kWave + lane]);  // past nz: not read below
        for (int32_t t = 0; t < m; ++t) {
            run += (double)__int_as_float(__builtin_amdgcn_readlane(av, t));
            pre[j] = lane == t ? run : pre[j];
        }
    }
    const double thr = beta * run;
    int32_t kept = nz;
#pragma unroll
    for (int j = J - 1; j >= 0; --j) {
        const uint64_t m = __ballot(j * kWave + lane < nz && pre[j] >= thr);
        if (m) kept = j * kWave + (int32_t)__ffsll((unsigned long long)m);
    }
    uint32_t bits = 0;
#pragma unroll
    for (int j = 0; j < J; ++j) bits |= (key[j] && rank[j] < kept) ? 1u << j : 0u;
    return bits;
}

// The fixed-point exponent of a query whose coarse sums are bounded by `bound`: the largest
// power of two keeping every partial sum within 2^30 in magnitude.
__device__ __forceinline__ int scale_exponent(float bound)
{
    int ex = 0;
    if (bound > 0.0f) {
        (void)frexpf(bound, &ex);  // bound < 2^ex
        ex = 30 - ex;
        ex = ex > 100 ? 100 : (ex < -100 ? -100 : ex);
    }
    return ex;
}

// A row of n <= 64 J entries at a: check, prune, scale and write its coarse terms.  Returns the
// malformed-row bits (nothing is written then).
template <int J>
__device__ __forceinline__ int prep_row(const DevQueries &q, int64_t n_cols, double beta,
                                        const DevCoarse &c, const float *term_max, int64_t row,
                                        int64_t a, int32_t n, PrepRow &r)
{
    const int lane = threadIdx.x & (kWave - 1);
    int32_t id[J];
    float v[J];
    uint64_t key[J];
    int bad = 0;
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const int32_t e = j * kWave + lane;
        id[j] = 0;
        v[j] = 0.0f;
        key[j] = 0;
        if (e < n) {
            id[j] = q.indices[a + e];
            v[j] = q.values[a + e];
            if (id[j] < 0 || id[j] >= n_cols) bad |= 2;
            if (e + 1 < n && q.indices[a + e + 1] <= id[j]) bad |= 4;
            if (!isfinite(v[j])) bad |= 8;
            if (v[j] != 0.0f)
                key[j] = ((uint64_t)__float_as_uint(fabsf(v[j])) << 32) | (0xFFFFFFFFu - (uint32_t)id[j]);
        }
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) bad |= __shfl_xor(bad, m, kWave);
    if (bad) return bad;
    uint32_t keep = 0;
    if (beta < 1.0) {
        keep = beta_mass_keep<J>(key, n, beta, r);
        wave_lds_sync();  // the keys give way to the kept entries
    } else {
#pragma unroll
        for (int j = 0; j < J; ++j) keep |= key[j] ? 1u << j : 0u;
    }
    // ordered compaction of the kept entries (ascending term id preserved)
    int32_t base = 0;
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const bool k = (keep >> j) & 1u;
        const uint64_t m = __ballot(k);
        if (k) {
            const int32_t p = base + (int32_t)lanes_below(m);
            r.id[p] = id[j];
            r.w[p] = v[j];
        }
        base += (int32_t)__popcll(m);
    }
    wave_lds_sync();
    float bound = 0.0f;
    for (int32_t i = lane; i < base; i += kWave) bound += fabsf(r.w[i]) * term_max[r.id[i]];
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) bound += __shfl_xor(bound, m, kWave);
    const int ex = scale_exponent(bound);
    const float scale = ldexpf(1.0f, ex);
    for (int32_t i = lane; i < base; i += kWave) {
        c.ct[a + i] = r.id[i];
        c.cw[a + i] = r.w[i] * scale;
    }
    if (lane == 0) {
        c.cn[row] = base;
        c.qinv[row] = ldexpf(1.0f, -ex);
    }
    return 0;
}

// The malformed-row bits of the entries [a, b).
__device__ int scan_row(const DevQueries &q, int64_t n_cols, int64_t a, int64_t b)
{
    const int lane = threadIdx.x & (kWave - 1);
    int bad = 0;
    for (int64_t e = a + lane; e < b; e += kWave) {
        int32_t id = q.indices[e];
        float v = q.values[e];
        if (id < 0 || id >= n_cols) bad |= 2;
        if (e + 1 < b && q.indices[e + 1] <= id) bad |= 4;
        if (!isfinite(v)) bad |= 8;
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) bad |= __shfl_xor(bad, m, kWave);
    return bad;
}

// A row [a, b) of more than kPrepRow entries, through global memory (sabs: FP64 scratch).
__device__ int prep_long_row(const DevQueries &q, int64_t n_cols, double beta, const DevCoarse &c,
                             const float *term_max, double *sabs, int64_t row, int64_t a, int64_t b)
{
    const int lane = threadIdx.x & (kWave - 1);
    if (const int bad = scan_row(q, n_cols, a, b)) return bad;
    int32_t r_keep = 0x7FFFFFFF;  // rank bound of kept entries
    if (beta < 1.0) {
        // rank of every non-zero entry in pi order; |x| placed at its rank
        int32_t nz = 0;
        for (int64_t e0 = a; e0 < b; e0 += kWave) {
            bool p = (e0 + lane < b) && q.values[e0 + lane] != 0.0f;
            nz += __popcll(__ballot(p));
        }
        for (int64_t e = a + lane; e < b; e += kWave) {
            float v = q.values[e];
            if (v == 0.0f) continue;
            float av = fabsf(v);
            int32_t id = q.indices[e];
            int32_t rank = 0;
            for (int64_t f = a; f < b; ++f) {
                float w = fabsf(q.values[f]);
                if (w == 0.0f) continue;
                int32_t jd = q.indices[f];
                rank += (w > av || (w == av && jd < id)) ? 1 : 0;
            }
            sabs[a + rank] = (double)av;
        }
        __threadfence();
        int32_t r = 0;
        if (lane == 0) {
            double mass = 0.0;
            for (int32_t t = 0; t < nz; ++t) mass += sabs[a + t];
            double thr = beta * mass;
            double run = 0.0;
            while (r < nz) {
                run += sabs[a + r];
                ++r;
                if (run >= thr) break;
            }
        }
        r_keep = __shfl(r, 0, kWave);
    }
    int32_t base = 0;
    for (int64_t e0 = a; e0 < b; e0 += kWave) {
        int64_t e = e0 + lane;
        bool keep = false;
        float v = 0.0f;
        int32_t id = 0;
        if (e < b) {
            v = q.values[e];
            id = q.indices[e];
            keep = v != 0.0f;
            if (keep && r_keep != 0x7FFFFFFF) {
                float av = fabsf(v);
                int32_t rank = 0;
                for (int64_t f = a; f < b; ++f) {
                    float w = fabsf(q.values[f]);
                    if (w == 0.0f) continue;
                    int32_t jd = q.indices[f];
                    rank += (w > av || (w == av && jd < id)) ? 1 : 0;
                }
                keep = rank < r_keep;
            }
        }
        uint64_t m = __ballot(keep);
        if (keep) {
            int32_t p = base + (int32_t)lanes_below(m);
            c.ct[a + p] = id;
            c.cw[a + p] = v;
        }
        base += __popcll(m);
    }
    float bound = 0.0f;
    for (int32_t i = lane; i < base; i += kWave)
        bound += fabsf(c.cw[a + i]) * term_max[c.ct[a + i]];
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) bound += __shfl_xor(bound, m, kWave);
    const int ex = scale_exponent(bound);
    const float scale = ldexpf(1.0f, ex);
    for (int32_t i = lane; i < base; i += kWave) c.cw[a + i] *= scale;
    if (lane == 0) {
        c.cn[row] = base;
        c.qinv[row] = ldexpf(1.0f, -ex);
    }
    return 0;
}

// One wave per query row.  Flags malformed rows (err[0] bits: 1 row pointers,
// 2 term id out of range, 4 ids not strictly ascending, 8 non-finite value,
// 16 more than kQueryHash / 2 entries), keeps the longest row in err[1]
// (err[0..3] must be zero where the grid has several workgroups), clears
// zero[0, n_zero) for the kernels that follow, and writes the coarse terms: the non-zero entries, cut to the beta-mass
// subvector when beta < 1 (entries ranked by |q| descending, ties by id;
// FP64 prefix sums in that order, the first prefix reaching beta * mass),
// with weights pre-multiplied by the query's fixed-point scale.
//
// Bound by latency: the row's entries are read once, one to eight per lane, and ranked, summed
// and compacted in the wave's registers and LDS.  At beta 0.8, 37 rows of 5 to 123 entries take
// 12 us and 7,000 rows of 35 take 19 us; ranking through global memory, summing on one lane and
// an atomic per row for the longest row took 93 and 242 us (86 us at beta 1, all of it atomics).
__global__ __launch_bounds__(kPrepWaves * kWave) void k_query_prep(DevQueries q, int64_t n_cols,
                                                                   double beta, DevCoarse c,
                                                                   const float *term_max,
                                                                   double *sabs, int32_t *err,
                                                                   uint32_t *zero, int64_t n_zero)
{
    __shared__ PrepRow s_row[kPrepWaves];
    __shared__ int32_t s_longest, s_bad;
    if (threadIdx.x == 0) s_longest = s_bad = 0;
    __syncthreads();
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n_zero;
         i += (int64_t)gridDim.x * blockDim.x)
        zero[i] = 0u;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = (int)uni((uint32_t)threadIdx.x / kWave);
    const int64_t row = (int64_t)blockIdx.x * kPrepWaves + wave;
    const bool live = row < q.n_rows;
    int64_t a = live ? q.indptr[row] : 0, b = live ? q.indptr[row + 1] : 0;
    int bad = 0;
    if (live && (a < 0 || b < a || b > q.nnz || (row == 0 && a != 0) ||
                 (row == q.n_rows - 1 && b != q.nnz)))
        bad |= 1;
    a = a < 0 ? 0 : (a > q.nnz ? q.nnz : a);
    b = b < a ? a : (b > q.nnz ? q.nnz : b);
    if (b - a > kQueryHash / 2) bad |= 16;
    PrepRow &r = s_row[wave];
    if (!live)
        ;
    else if (bad)
        bad |= scan_row(q, n_cols, a, b);
    else if (b - a <= kWave)
        bad = prep_row<1>(q, n_cols, beta, c, term_max, row, a, (int32_t)(b - a), r);
    else if (b - a <= 2 * kWave)
        bad = prep_row<2>(q, n_cols, beta, c, term_max, row, a, (int32_t)(b - a), r);
    else if (b - a <= 4 * kWave)
        bad = prep_row<4>(q, n_cols, beta, c, term_max, row, a, (int32_t)(b - a), r);
    else if (b - a <= kPrepRow)
        bad = prep_row<kPrepRow / kWave>(q, n_cols, beta, c, term_max, row, a, (int32_t)(b - a), r);
    else
        bad = prep_long_row(q, n_cols, beta, c, term_max, sabs, row, a, b);
    if (live && lane == 0) {
        if (bad) {
            atomicOr(&s_bad, bad);
            c.cn[row] = 0;
            c.qinv[row] = 1.0f;
        } else {
            atomicMax(&s_longest, (int32_t)(b - a));
        }
    }
    // flags and the longest row (sizes the rerank table): a lone workgroup writes them (and the
    // two retry counts behind them); else one device atomic per workgroup, and none where the value
    // is already reached (an atomic of every row on one word cost 12 ns each)
    __syncthreads();
    if (threadIdx.x != 0) return;
    if (gridDim.x == 1) {
        err[0] = s_bad;
        err[1] = s_longest;
        err[2] = err[3] = 0;
        return;
    }
    if (s_bad) atomicOr(err, s_bad);
    if (__hip_atomic_load(err + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < s_longest)
        atomicMax(err + 1, s_longest);
}

// ------------------------------------------------------------------ accumulate
// Posting values: raw bits of one aligned 4-posting group, decoded after
// every load of the step has been issued.
template <int VT> struct Val;
template <> struct Val<0> {  // FP32
    using Raw = uint4;
    static __device__ __forceinline__ Raw load(const void *p, uint64_t g)
    {
        return reinterpret_cast<const uint4 *>(p)[g];
    }
    static __device__ __forceinline__ void decode(const Raw &r, float (&v)[4])
    {
        v[0] = __uint_as_float(r.x);
        v[1] = __uint_as_float(r.y);
        v[2] = __uint_as_float(r.z);
        v[3] = __uint_as_float(r.w);
    }
    // w * x_p rounded to FP32
    static __device__ __forceinline__ float prod(const Raw &r, int p, float w)
    {
        const uint32_t b = p == 0 ? r.x : (p == 1 ? r.y : (p == 2 ? r.z : r.w));
        return w * __uint_as_float(b);
    }
};
template <> struct Val<1> {  // FP16
    using Raw = uint2;
    static __device__ __forceinline__ Raw load(const void *p, uint64_t g)
    {
        return reinterpret_cast<const uint2 *>(p)[g];
    }
    static __device__ __forceinline__ float h2f(uint32_t h)
    {
        return (float)__builtin_bit_cast(_Float16, (uint16_t)h);
    }
    static __device__ __forceinline__ void decode(const Raw &r, float (&v)[4])
    {
        v[0] = h2f(r.x & 0xFFFFu);
        v[1] = h2f(r.x >> 16);
        v[2] = h2f(r.y & 0xFFFFu);
        v[3] = h2f(r.y >> 16);
    }
    // w * x_p rounded to FP32: the FP16 value widens exactly, and a fused
    // multiply-add with a +0 addend rounds the product once, as a multiply
    // does (the sign of a zero product is lost, which the integer conversion
    // that follows ignores); one mixed-precision FMA does both steps.
    static __device__ __forceinline__ float prod(const Raw &r, int p, float w)
    {
        const uint32_t word = p < 2 ? r.x : r.y;
        const uint32_t bits = (p & 1) ? (word >> 16) : (word & 0xFFFFu);
        return __builtin_fmaf(w, h2f(bits), 0.0f);
    }
};
template <> struct Val<2> {  // BF16
    using Raw = uint2;
    static __device__ __forceinline__ Raw load(const void *p, uint64_t g)
    {
        return reinterpret_cast<const uint2 *>(p)[g];
    }
    static __device__ __forceinline__ void decode(const Raw &r, float (&v)[4])
    {
        v[0] = __uint_as_float(r.x << 16);
        v[1] = __uint_as_float(r.x & 0xFFFF0000u);
        v[2] = __uint_as_float(r.y << 16);
        v[3] = __uint_as_float(r.y & 0xFFFF0000u);
    }
    static __device__ __forceinline__ float prod(const Raw &r, int p, float w)
    {
        const uint32_t word = p < 2 ? r.x : r.y;
        return w * __uint_as_float((p & 1) ? (word & 0xFFFF0000u) : (word << 16));
    }
};

// Emit the scores of one query row segment that reach the threshold: each
// lane holds NV scores of consecutive documents starting at m0.
template <int NV>
__device__ __forceinline__ void emit_candidates(const float (&sv)[NV], const bool (&ok)[NV],
                                                int64_t doc0, uint32_t *cnt, uint64_t *out,
                                                int64_t cap)
{
    const int lane = threadIdx.x & (kWave - 1);
    uint64_t bal[NV];
    uint32_t tot = 0;
#pragma unroll
    for (int p = 0; p < NV; ++p) {
        bal[p] = __ballot(ok[p]);
        tot += (uint32_t)__popcll(bal[p]);
    }
    uint32_t b0 = 0;
    if (lane == 0) b0 = atomicAdd(cnt, tot);
    b0 = __shfl(b0, 0, kWave);
#pragma unroll
    for (int p = 0; p < NV; ++p) {
        if (ok[p]) {
            const uint64_t pos = (uint64_t)b0 + lanes_below(bal[p]);
            if (pos < (uint64_t)cap) out[pos] = make_key(sv[p], (uint32_t)(doc0 + p));
        }
        b0 += (uint32_t)__popcll(bal[p]);
    }
}

// Smallest fixed-point sum a with (float)a * qinv >= th, as an int64 (2^31 if
// no int32 sum reaches th).  (float)a * qinv is non-decreasing in a, so the
// scores at or above th are exactly the sums at or above this bound.
__device__ int64_t sum_threshold(float th, float qinv)
{
    auto reaches = [&](int64_t a) { return (float)(int32_t)a * qinv >= th; };
    if (!reaches(INT32_MAX)) return (int64_t)INT32_MAX + 1;
    int64_t lo = INT32_MIN, hi = INT32_MAX;  // invariant: reaches(hi)
    if (reaches(lo)) return lo;
    while (hi - lo > 1) {                     // invariant: !reaches(lo)
        const int64_t mid = lo + (hi - lo) / 2;
        if (reaches(mid)) hi = mid; else lo = mid;
    }
    return hi;
}

// The same bound by one wave, clamped to INT32_MAX: 64 probes a round.
__device__ __forceinline__ int32_t sum_threshold_wave(float th, float qinv)
{
    const int lane = threadIdx.x & (kWave - 1);
    auto reaches = [&](int64_t a) { return (float)(int32_t)a * qinv >= th; };
    if (!reaches(INT32_MAX)) return INT32_MAX;
    int64_t lo = INT32_MIN, hi = INT32_MAX;
    if (reaches(lo)) return INT32_MIN;
    while (hi - lo > 1) {  // invariants: !reaches(lo), reaches(hi); probes ascend inside (lo, hi)
        const int64_t base = lo + 1, span = hi - lo - 1;
        const uint64_t r = __ballot(reaches(base + span * lane / kWave));
        const int f = r ? __ffsll((unsigned long long)r) - 1 : kWave;
        if (f > 0) lo = base + span * (f - 1) / kWave;
        if (f < kWave) hi = base + span * f / kWave;
    }
    return (int32_t)hi;
}

// Decode a pair-packed 64-bit score word into the two 32-bit sums it holds:
// the word is H * 2^32 + L (exactly, modulo 2^64) with |L|, |H| < 2^31.
__device__ __forceinline__ void unpack_pair(uint32_t wlo, uint32_t whi, int32_t &l, int32_t &h)
{
    l = (int32_t)wlo;
    h = (int32_t)(whi + (l < 0 ? 1u : 0u));
}

// One workgroup = a batch of B >= 2 query slots x a contiguous run of tiles.  The
// batch's (query, term) entries are first merged into one ascending list of
// distinct terms, each with a weight per query (zero where the query lacks
// the term), so a list I_{term, tile} shared by several queries of the batch
// is read once.  Then, for every tile: the score rows (the window's distance
// array of Sec. 3.3.1, one per query) are cleared in LDS; the tile's lists of
// all merged terms (each padded to whole 4-posting groups with zero values)
// are cut into chunks of up to 64 groups, and each wave takes a contiguous
// share of the chunks, several chunks in flight: one group per lane, so a
// chunk's list, weights and base address are wave-uniform (scalar registers)
// and a lane only adds its group's offset.  Every posting adds w_b * x to
// query b's score of its document (Alg. 2: product, then accumulate).
//
// Scores are 32-bit fixed point: weights arrive multiplied by the query's
// power-of-two scale and each product is truncated once to an integer, so
// the sums are exact and independent of the order of the adds; different
// terms can hit one document concurrently, so the adds are LDS atomics, and
// integer LDS atomics run many times faster than float ones on this chip.
// For B >= 2 the rows of queries 2q and 2q+1 are interleaved into one 64-bit
// word per document holding H * 2^32 + L, so one 64-bit atomic updates both
// (the sums stay within +-2^30, so both halves decode exactly).
//
// Finally each row is either sampled (per-thread maxima, for the candidate
// threshold) or every score at or above the query's threshold is appended to
// its candidate list.
template <int VT, int B, bool SAMPLE>
__global__ __launch_bounds__(kAccThreads) __attribute__((amdgpu_waves_per_eu(6))) void k_accumulate(
    DevIndex ix, DevQueries q, DevCoarse c, DevSlots slots,
    int32_t n_sample, float *maxima, const float *theta, uint32_t *count, uint64_t *cand,
    int64_t cap, int32_t tiles_per_wg, int32_t eb)
{
    constexpr int NT = kAccThreads, NW = NT / kWave;
    const int32_t n_slots = slots.n;
    const int EB = eb;  // entries merged per pass: a power of two, at most NT
    constexpr int NP = B / 2;            // score words per document
    constexpr int KU = VT == 0 ? 4 : 8;  // chunks in flight per wave
    static_assert(B >= 2 && B % 2 == 0, "one query per workgroup runs in k_accumulate1");
    static_assert(kEntryBlock <= NT, "at most one merged entry per thread");
    extern __shared__ __align__(16) unsigned char smem[];
    const int T = ix.tile_stride;
    // score rows: uint64 [NP][T], B * T * 4 bytes
    unsigned char *A = smem;
    // the merged term list (u_term / u_w, EB entries)
    int32_t *u_term = reinterpret_cast<int32_t *>(smem + (size_t)B * T * 4);
    float *u_w = reinterpret_cast<float *>(u_term + EB);  // [EB][B]
    unsigned char *region = reinterpret_cast<unsigned char *>(u_w + (size_t)EB * B);
    uint64_t *keys = reinterpret_cast<uint64_t *>(region);                 // merge phase
    uint32_t *flag = reinterpret_cast<uint32_t *>(keys + EB);              // merge phase
    uint32_t *l_base = reinterpret_cast<uint32_t *>(region);               // tile phase
    uint32_t *l_end = l_base + EB;
    uint32_t *l_cp = l_end + EB;                                           // EB + 1 (+3)
    float *l_w = reinterpret_cast<float *>(l_cp + EB + 4);                 // [EB][B]
    __shared__ int64_t s_qa[B];
    __shared__ int32_t s_qpre[B + 1];
    __shared__ int32_t s_slot[B];
    __shared__ float s_qinv[B];
    __shared__ uint32_t s_wsum[NW];
    __shared__ int32_t s_nu;
    __shared__ uint32_t s_wl[NW];  // list holding each wave's first chunk
    __shared__ int32_t s_thr[B];   // per query: smallest sum at or above its threshold
    __shared__ int32_t s_none[B];  // per query: no sum reaches the threshold
    __shared__ int32_t s_imp[B];   // per query: threshold <= 0, zero sums left implicit

    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = (int)uni((uint32_t)tid / kWave);  // uniform per wave: keeps chunk bookkeeping scalar
    const int32_t batch = blockIdx.x;
    if (tid == 0) {
        int32_t acc = 0;
        for (int b = 0; b < B; ++b) {
            const int32_t s = batch * B + b;
            int32_t n = 0;
            int64_t qa = 0;
            float qinv = 1.0f;
            if (s < n_slots) {
                const int32_t row = slots.row(s);
                qa = q.indptr[row];
                n = c.cn[row];
                qinv = c.qinv[row];
            }
            s_slot[b] = s < n_slots ? s : -1;
            s_qinv[b] = qinv;
            s_qa[b] = qa;
            s_qpre[b] = acc;
            acc += n;
        }
        s_qpre[B] = acc;
    }
    if (!SAMPLE && tid < B) {
        const int32_t s2 = batch * B + tid;
        const int64_t a = s2 < n_slots ? sum_threshold(theta ? theta[s2] : -INFINITY, c.qinv[slots.row(s2)])
                                       : (int64_t)INT32_MAX + 1;
        s_none[tid] = a > INT32_MAX;
        s_thr[tid] = a > INT32_MAX ? INT32_MAX : (int32_t)a;
        const float th = s2 < n_slots ? (theta ? theta[s2] : -INFINITY) : 1.0f;
        s_imp[tid] = th <= 0.0f && th != -INFINITY;
    }
    __syncthreads();
    const int32_t n_e = s_qpre[B];
    const int32_t n_blocks = (n_e + EB - 1) / EB;

    // Merge entries [e0, e0 + EB) of the batch into u_term / u_w (s_nu terms).
    auto merge = [&](int32_t e0) {
        const int32_t ne = min(EB, n_e - e0);
        int P = 1;
        while (P < ne) P <<= 1;
        if (tid < P) {
            uint64_t key = ~0ull;
            if (tid < ne) {
                const int32_t e = e0 + tid;
                int b = 0;
                while (b + 1 < B && s_qpre[b + 1] <= e) ++b;
                key = ((uint64_t)(uint32_t)c.ct[s_qa[b] + (e - s_qpre[b])] << 32) | (uint32_t)tid;
            }
            keys[tid] = key;
        }
        __syncthreads();
        for (int kk = 2; kk <= P; kk <<= 1) {
            for (int j = kk >> 1; j > 0; j >>= 1) {
                if (tid < P) {
                    const int ij = tid ^ j;
                    if (ij > tid) {
                        const uint64_t x = keys[tid], y = keys[ij];
                        const bool up = (tid & kk) == 0;
                        if (up ? (x > y) : (x < y)) {
                            keys[tid] = y;
                            keys[ij] = x;
                        }
                    }
                }
                __syncthreads();
            }
        }
        const uint32_t fresh =
            (tid < ne && (tid == 0 || (keys[tid] >> 32) != (keys[tid - 1] >> 32))) ? 1u : 0u;
        uint32_t nu;
        const uint32_t ex = block_excl_scan<NT>(fresh, s_wsum, nu);
        for (int i = tid; i < (int)nu * B; i += NT) u_w[i] = 0.0f;
        if (tid < EB) flag[tid] = ex + fresh;  // 1-based merged index of this sorted entry's term
        if (tid == 0) s_nu = (int32_t)nu;
        __syncthreads();
        if (tid < ne) {
            const uint64_t key = keys[tid];
            const int32_t u = (int32_t)flag[tid] - 1;
            const int32_t e = e0 + (int32_t)(key & 0xFFFFFFFFu);
            int b = 0;
            while (b + 1 < B && s_qpre[b + 1] <= e) ++b;
            if (fresh) u_term[u] = (int32_t)(key >> 32);
            u_w[u * B + b] = c.cw[s_qa[b] + (e - s_qpre[b])];
        }
        __syncthreads();
    };

    if (n_blocks == 1) merge(0);
    const int64_t n_tile_iter = SAMPLE ? n_sample : ix.n_tiles;
    using Raw = typename Val<VT>::Raw;

    // With one merged block, each thread prefetches its term's list bounds of
    // the next tile while the current tile accumulates.
    uint32_t pre_lo = 0, pre_hi = 0;
    bool have_pre = false;
    // Workgroup y sweeps tiles [y R, (y + 1) R).  Workgroups are dispatched batch
    // fastest, so those resident together walk the same tiles at about the
    // same pace and share the tiles' lists in L2.
    const int64_t ti_beg = (int64_t)blockIdx.y * tiles_per_wg;
    const int64_t ti_end = min(n_tile_iter, ti_beg + tiles_per_wg);
    // the score rows start cleared; reading a tile's rows clears them again
    {
        int4 *A4 = reinterpret_cast<int4 *>(A);
        for (int i = tid; i < B * T / 4; i += NT) A4[i] = make_int4(0, 0, 0, 0);
    }
    __syncthreads();
    for (int64_t ti = ti_beg; ti < ti_end; ++ti) {
        const int64_t t = SAMPLE ? (ti * ix.n_tiles / n_sample) : ti;
        const int64_t d0 = ix.tile_doc[t];
        const int32_t len = (int32_t)(ix.tile_doc[t + 1] - d0);
        const uint64_t G0 = (uint64_t)ix.tile_post[t] >> 2;  // first 4-posting group of the tile
        const uint32_t *toff = ix.term_goff + (size_t)t * (size_t)(ix.n_cols + 1);

        for (int32_t blk = 0; blk < n_blocks; ++blk) {
            if (n_blocks > 1) merge(blk * EB);
            const int32_t nu = s_nu;
            // list (term, tile) = groups [gs, gs + ng) of the tile, cut into chunks
            // of kChunk groups; the non-empty lists are compacted in term order
            // with the index of their first chunk
            uint32_t gs = 0, ng = 0;
            if (tid < nu) {
                const int32_t term = u_term[tid];
                const uint32_t lo = have_pre ? pre_lo : toff[term];
                const uint32_t hi = have_pre ? pre_hi : toff[term + 1];
                gs = lo & kGoffMask;
                ng = (hi & kGoffMask) - gs;
            }
            const uint32_t nch = (ng + kChunk - 1) / kChunk;
            uint32_t total;
            // low 20 bits: chunks before this list; high bits: non-empty lists before it
            const uint32_t ex = block_excl_scan<NT>(nch | (nch ? (1u << 20) : 0u), s_wsum, total);
            // the scan's barriers order these writes after the merge-phase reads
            if (nch) {
                // chunk ci of list li covers groups [l_base + 64 ci, min(+64, l_end)) of
                // the tile (l_base wraps below zero as an unsigned number)
                const uint32_t li = ex >> 20;
                l_base[li] = gs - (ex & 0xFFFFFu) * (uint32_t)kChunk;
                l_end[li] = gs + ng;
                l_cp[li] = ex & 0xFFFFFu;
#pragma unroll
                for (int b = 0; b < B; ++b) l_w[li * B + b] = u_w[tid * B + b];
            }
            const uint32_t n_list = total >> 20, n_chunk = total & 0xFFFFFu;
            if (tid == 0) l_cp[n_list] = n_chunk;
            // wave w takes chunks [n_chunk w / NW, n_chunk (w + 1) / NW)
            if (nch) {
                const uint32_t c0l = ex & 0xFFFFFu;
#pragma unroll
                for (int w2 = 0; w2 < NW; ++w2) {
                    const uint32_t cb = (uint32_t)(((uint64_t)n_chunk * (uint32_t)w2) / NW);
                    if (cb >= c0l && cb < c0l + nch) s_wl[w2] = ex >> 20;
                }
            }
            have_pre = false;
            if (n_blocks == 1) {
                const int64_t tn = ti + 1;
                if (tn < ti_end) {
                    have_pre = true;
                    if (tid < nu) {
                        const int64_t t2 = SAMPLE ? (tn * ix.n_tiles / n_sample) : tn;
                        const uint32_t *toff2 = ix.term_goff + (size_t)t2 * (size_t)(ix.n_cols + 1);
                        const int32_t term = u_term[tid];
                        pre_lo = toff2[term];
                        pre_hi = toff2[term + 1];
                    }
                }
            }
            __syncthreads();

            // This wave's contiguous share of the chunks.  One chunk = up to 64
            // consecutive groups of one list, one group (4 postings) per lane, so a
            // chunk's list, weights and base address are wave-uniform.  The wave
            // reads the bounds of 64 consecutive lists at once (one per lane); a
            // chunk finds its list among them by a ballot over the lists' first
            // chunks and takes the list's fields by lane broadcast, so KU chunks'
            // loads leave back to back even where they cross lists.
            const uint32_t c_beg = (uint32_t)(((uint64_t)n_chunk * (uint32_t)wave) / NW);
            const uint32_t c_end = (uint32_t)(((uint64_t)n_chunk * (uint32_t)(wave + 1)) / NW);
            if (c_beg < c_end) {
                // the tile's groups, addressed by 32-bit byte offsets (a tile holds at
                // most kTileGroupsMax groups; the arrays end with kTailSlots zero postings)
                const gbytes pd_t = uni_ptr(
                    reinterpret_cast<const unsigned char *>(ix.post_doc) + G0 * sizeof(uint2));
                const gbytes pv_t = uni_ptr(
                    reinterpret_cast<const unsigned char *>(ix.post_val) + G0 * sizeof(Raw));
                uint32_t lp0 = uni(s_wl[wave]);  // list of chunk c
                for (uint32_t c = c_beg; c < c_end;) {
                    const uint32_t lw = lp0 + (uint32_t)lane;
                    const uint32_t cpn = lw + 1 <= n_list ? l_cp[lw + 1] : 0xFFFFFFFFu;
                    uint32_t basel = 0, endl = 0;
                    float wl[B];
#pragma unroll
                    for (int b = 0; b < B; ++b) wl[b] = 0.0f;
                    if (lw < n_list) {
                        basel = l_base[lw];
                        endl = l_end[lw];
#pragma unroll
                        for (int b = 0; b < B; ++b) wl[b] = l_w[lw * B + b];
                    }
                    // the window's chunks lie in lists lp0 .. lp0 + 63
                    const uint32_t c_win = min(c_end, c + (uint32_t)kWave);
                    for (uint32_t cs = c; cs < c_win; cs += KU) {
                        uint2 ids[KU];
                        Raw raw[KU];
                        uint32_t nl[KU];
                        int32_t kl[KU];
                        // Loads are unconditional, so they leave back to back: lane l reads
                        // group g0 + l even past its chunk's end (at most 63 groups past the
                        // end of a list of this tile: inside the arrays), and a slot past the
                        // window reads the tile's first groups; those lanes add nothing.
#pragma unroll
                        for (int i = 0; i < KU; ++i) {
                            const uint32_t ci = cs + (uint32_t)i;
                            uint32_t g0 = 0, n = 0;
                            int32_t k = 0;
                            if (ci < c_win) {  // wave-uniform
                                k = (int32_t)__popcll(__ballot(cpn <= ci));
                                g0 = (uint32_t)__builtin_amdgcn_readlane((int)basel, k) +
                                     ci * (uint32_t)kChunk;
                                n = min((uint32_t)kChunk,
                                        (uint32_t)__builtin_amdgcn_readlane((int)endl, k) - g0);
                            }
                            kl[i] = k;
                            nl[i] = n;
                            const uint32_t gi = g0 + (uint32_t)lane;
                            load_at(pd_t, gi * (uint32_t)sizeof(uint2), ids[i]);
                            load_at(pv_t, gi * (uint32_t)sizeof(Raw), raw[i]);
                        }
#pragma unroll
                        for (int i = 0; i < KU; ++i) {
                            if ((uint32_t)lane >= nl[i]) continue;
                            float w[B];
#pragma unroll
                            for (int b = 0; b < B; ++b)
                                w[b] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wl[b]), kl[i]));
                            // byte offsets of the documents' 32-bit score words
                            const uint32_t d4[4] = {ids[i].x & 0xFFFFu, ids[i].x >> 16,
                                                    ids[i].y & 0xFFFFu, ids[i].y >> 16};
                            float v[4];
                            Val<VT>::decode(raw[i], v);
                            unsigned char *A8 = A;
#pragma unroll
                            for (int qp = 0; qp < NP; ++qp) {
                                const float w0 = w[2 * qp], w1 = w[2 * qp + 1];
                                if (w0 == 0.0f && w1 == 0.0f) continue;
#pragma unroll
                                for (int p = 0; p < 4; ++p) {
                                    const int32_t lo = (int32_t)(w0 * v[p]);
                                    const int32_t hi = (int32_t)(w1 * v[p]);
                                    const uint32_t hw = (uint32_t)hi + (uint32_t)(lo >> 31);
                                    const uint64_t add = ((uint64_t)hw << 32) | (uint32_t)lo;
                                    uint64_t *dst = reinterpret_cast<uint64_t *>(
                                        A8 + (size_t)qp * T * 8 + 2u * d4[p]);
                                    __hip_atomic_fetch_add(dst, add, __ATOMIC_RELAXED,
                                                           __HIP_MEMORY_SCOPE_WORKGROUP);
                                }
                            }
                        }
                    }
                    // list of the next window's first chunk
                    lp0 += c_win < c_end ? (uint32_t)__popcll(__ballot(cpn <= c_win)) : 0u;
                    c = c_win;
                }
            }
            __syncthreads();
        }

        // ---- read the rows: sample maxima or emit every score at or above the
        // query's threshold, compared as the integer sum against the smallest sum
        // that reaches the threshold
        uint64_t *A64 = reinterpret_cast<uint64_t *>(A);
        for (int qp = 0; qp < NP; ++qp) {
            const int32_t sl0 = s_slot[2 * qp], sl1 = s_slot[2 * qp + 1];
            const bool any0 = sl0 >= 0 && (SAMPLE || !s_none[2 * qp]);
            const bool any1 = sl1 >= 0 && (SAMPLE || !s_none[2 * qp + 1]);
            uint64_t *row = A64 + (size_t)qp * T;
            if (!any0 && !any1) {
                for (int m = tid * 2; m < len; m += NT * 2)
                    *reinterpret_cast<int4 *>(row + m) = fresh_zero4();
                continue;
            }
            const float qi0 = s_qinv[2 * qp], qi1 = s_qinv[2 * qp + 1];
            if (SAMPLE) {
                int32_t m0 = INT32_MIN, m1 = INT32_MIN;
                for (int m = tid; m < len; m += NT) {
                    const uint64_t wd = row[m];
                    row[m] = 0ull;
                    int32_t l, h;
                    unpack_pair((uint32_t)wd, (uint32_t)(wd >> 32), l, h);
                    m0 = max(m0, l);
                    m1 = max(m1, h);
                }
                if (sl0 >= 0)
                    maxima[((size_t)sl0 * n_sample + ti) * NT + tid] = tid < len ? (float)m0 * qi0 : -INFINITY;
                if (sl1 >= 0)
                    maxima[((size_t)sl1 * n_sample + ti) * NT + tid] = tid < len ? (float)m1 * qi1 : -INFINITY;
            } else {
                const int32_t th0 = s_thr[2 * qp], th1 = s_thr[2 * qp + 1];
                const bool imp0 = s_imp[2 * qp], imp1 = s_imp[2 * qp + 1];
                for (int base = wave * 128; base < len; base += NW * 128) {
                    const int m0 = base + lane * 2;
                    int4 r = make_int4(0, 0, 0, 0);
                    if (m0 < len) {
                        r = *reinterpret_cast<const int4 *>(row + m0);
                        *reinterpret_cast<int4 *>(row + m0) = fresh_zero4();
                    }
                    int32_t l0, h0, l1, h1;
                    unpack_pair((uint32_t)r.x, (uint32_t)r.y, l0, h0);
                    unpack_pair((uint32_t)r.z, (uint32_t)r.w, l1, h1);
                    // threshold <= 0: every nonzero sum, negative ones included, so that
                    // the finalize kernel may take each document left out as a zero
                    const bool oa[2] = {any0 && m0 < len && (imp0 ? l0 != 0 : l0 >= th0),
                                        any0 && m0 + 1 < len && (imp0 ? l1 != 0 : l1 >= th0)};
                    const bool ob[2] = {any1 && m0 < len && (imp1 ? h0 != 0 : h0 >= th1),
                                        any1 && m0 + 1 < len && (imp1 ? h1 != 0 : h1 >= th1)};
                    if (__ballot(oa[0] || oa[1] || ob[0] || ob[1]) == 0) continue;
                    const float a[2] = {(float)l0 * qi0, (float)l1 * qi0};
                    const float b2[2] = {(float)h0 * qi1, (float)h1 * qi1};
                    if (sl0 >= 0)
                        emit_candidates<2>(a, oa, d0 + m0, count + sl0, cand + (size_t)sl0 * cap, cap);
                    if (sl1 >= 0)
                        emit_candidates<2>(b2, ob, d0 + m0, count + sl1, cand + (size_t)sl1 * cap, cap);
                }
            }
        }
        __syncthreads();
    }
}

// The items of a launch: tile-major, `run` slots each.  Queue x of a queue-fed launch holds those of
// tiles x, x + queues, ...
struct AccItems {
    int64_t n;           // items in all
    int32_t run, groups; // slots per item, items per tile
    uint32_t tiles;
    int32_t queues;
};
// The arguments of a one-query launch.  They are read from the kernel-argument segment where they
// are used (acc_args), through the scalar cache: held in registers across the items they took some
// forty scalar registers, and what did not fit was spilled to vector lanes inside the loops.
struct AccArgs {
    DevIndex ix;
    DevQueries q;
    DevCoarse c;
    DevSlots slots;
    int32_t n_sample;
    float *maxima;
    const float *theta;
    const int32_t *sum_min;
    uint32_t *count;
    uint64_t *cand;
    int64_t cap;
    AccItems items;
    unsigned long long *head;
};
using acc_args_t = const AccArgs __attribute__((address_space(4))) *;
__device__ __forceinline__ acc_args_t acc_args()
{
    acc_args_t p = (acc_args_t)__builtin_amdgcn_kernarg_segment_ptr();
    __asm__ volatile("" : "+s"(p));  // a fresh pointer: loads through it are not kept from earlier
    return p;
}

// The single-query form of k_accumulate (same scores, same read-out).  One work item: the query
// slots [s0, s1), at most 64 of them, one after another over one tile.  The tile's data are then
// fixed for the item, and the workgroups resident together hold the items of few tiles, whose lists
// stay in L2 (1.4 MB a tile at 8.8M documents and alpha 0.5) while every query of the call passes over
// them: 7,000 queries at 8.8M documents read 13.5 GB beyond L2 and take 48.3 ms, where items of one
// query over a run of 12 tiles, drifting apart within the run, read 292 GB and took 50.6 ms; 1,000
// queries over 1M documents 0.90 against 1.11 ms.  (46.0 and 0.82 ms with what is described below.)
//
// The query's terms are taken 64 at a time (a segment, one list per lane), and a wave-wide
// prefix sum over the lists' chunk counts numbers the segment's chunks.  The
// waves then take batches of KU consecutive chunks: wave w's first batch of a
// segment is fixed (chunks w KU to w KU + KU - 1, so its loads leave at once),
// the next ones come from the segment's counter in LDS (one atomic by the
// wave's first lane, taken while the current batch's loads are in flight), so
// they finish the query together however unevenly the lists' lengths and the
// adds' bank conflicts fall; the counters are reset between the query's two
// barriers.  One wave lays out a query's first segment for all, a query ahead; of a longer query
// every wave lays out the further segments itself.
//
// The score row must be all zero on entry unless clear_row (the read-out of every query clears
// what its adds touched, so it is all zero again on return).  last() is called once, as the
// item's last query starts.
template <int VT, bool SAMPLE, typename Last>
__device__ __forceinline__ void accumulate1_item(int64_t ti, int32_t s0, int32_t s1, bool clear_row,
                                                 Last last)
{
    constexpr int NT = kAccThreads, NW = NT / kWave;
    constexpr int KU = VT == 0 ? 3 : 5;  // chunks per batch of a wave
    extern __shared__ __align__(16) unsigned char smem[];
    int32_t *A32 = reinterpret_cast<int32_t *>(smem);  // the query's score row [tile_stride]
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = (int)uni((uint32_t)tid / kWave);
    using Raw = typename Val<VT>::Raw;
    const acc_args_t g = acc_args();
    // the item's queries, one per lane: coarse terms, scale, least sum at the threshold
    const int32_t m = s1 - s0;
    int64_t r_qa = 0;
    int32_t r_n = 0, r_th = INT32_MIN;  // r_n bit 16: threshold <= 0, zero sums left implicit
    float r_qinv = 1.0f;
    const bool every = !SAMPLE && !g->theta;  // no threshold: every document is a candidate
    if (lane < m) {
        const int32_t row = g->slots.rows ? g->slots.rows[s0 + lane] : g->slots.row0 + s0 + lane;
        r_qa = g->q.indptr[row];
        r_n = g->c.cn[row];
        r_qinv = g->c.qinv[row];
        if (!SAMPLE && !every) {
            const float tv = g->theta[s0 + lane];
            r_th = g->sum_min[s0 + lane];
            r_n |= (tv <= 0.0f && tv != -INFINITY) ? 1 << 16 : 0;
        }
    }
    const int64_t t = SAMPLE ? (ti * g->ix.n_tiles / g->n_sample) : ti;
    const int64_t d0 = uni64(g->ix.tile_doc[t]);
    const int32_t len = (int32_t)uni((uint32_t)(g->ix.tile_doc[t + 1] - d0));
    const int64_t p0 = uni64(g->ix.tile_post[t]);
    const uint64_t G0 = (uint64_t)p0 >> 2;  // first 4-posting group of the tile
    const uint32_t n_groups = uni((uint32_t)((g->ix.tile_post[t + 1] - p0) >> 2));
    const uint32_t *toff = g->ix.term_goff + (size_t)t * (size_t)(g->ix.n_cols + 1);
    const int32_t *ct = g->c.ct;
    const float *cw = g->c.cw;
    // the tile's groups, addressed by 32-bit byte offsets (a tile holds at most
    // kTileGroupsMax groups; the arrays end with kTailSlots zero postings)
    const gbytes pd_t =
        uni_ptr(reinterpret_cast<const unsigned char *>(g->ix.post_doc) + G0 * sizeof(uint2));
    const gbytes pv_t =
        uni_ptr(reinterpret_cast<const unsigned char *>(g->ix.post_val) + G0 * sizeof(Raw));

    // the score row starts cleared; reading a query's row clears it again
    if (clear_row) {
        int4 *A4 = reinterpret_cast<int4 *>(smem);
        for (int i = tid; i < g->ix.tile_stride / 4; i += NT) A4[i] = make_int4(0, 0, 0, 0);
    }
    // The waves take batches of KU chunks of a segment from the segment's counter, so that
    // they reach the query's barrier together; wave w's first batch of a segment is chunks
    // [w KU, (w + 1) KU), so the counters start past the NW first batches.
    constexpr uint32_t kFirstTaken = (uint32_t)(NW * KU);
    __shared__ uint32_t s_next[kMaxSeg];
    for (int i = tid; i < kMaxSeg; i += NT) s_next[i] = kFirstTaken;
    // Candidates of the item's queries, {sum, query in the item, document in the tile}, held in LDS
    // until the item ends or the buffer is half full, then placed by one device atomic per query.
    // A read-out that takes its places in the candidate list from the device counter waits for
    // that atomic between the query's barriers, and the workgroups of few queries queue up at
    // their counters: 37 queries over 24 tiles 163 us, 30 us from the buffer; one query over 704
    // tiles 32 and 25 us.
    // s_cand_n counts them (and those past the buffer's end), query by query: query i's end at lane
    // i's r_end.
    __shared__ uint64_t s_cand[kCandBuf];
    __shared__ uint32_t s_cand_n, s_place[kWave];
    uint32_t r_end = 0;
    int32_t i_flush = 0;  // first query whose candidates are in the buffer
    if (tid == 0) s_cand_n = 0;

    // first segment of query i (none past the item): lane l holds term l
    auto terms = [&](int32_t i, int32_t &term, float &w) {
        term = 0;
        w = 0.0f;
        if (i >= m) return;  // uniform
        const int32_t n = __builtin_amdgcn_readlane(r_n, i) & 0xFFFF;
        const int64_t qa = readlane64(r_qa, i);
        if (lane < n) {
            term = (ct + qa)[lane];
            w = (cw + qa)[lane];
        }
    };
    // The lists of a segment, one per lane, as numbered chunks: list l holds chunks [incl - nch,
    // incl) of the segment, its chunk 0 would start at group basel, it ends at group endl.
    struct Lists {
        uint32_t cpn, basel, endl;
        float w;
    };
    auto plan = [&](uint32_t lo, uint32_t hi, bool live, float w) {
        const uint32_t gs = lo & kGoffMask, ng = live ? (hi & kGoffMask) - gs : 0u;
        const uint32_t nch = (ng + kChunk - 1) / kChunk;
        Lists r;
        r.cpn = wave_incl_scan(nch);
        r.basel = gs - (r.cpn - nch) * (uint32_t)kChunk;
        r.endl = gs + ng;
        r.w = w;
        return r;
    };
    // One wave, the planner, lays out the first segment of the next query while this one is
    // scored and leaves it in LDS; it also keeps the loads ahead: the next query's list bounds, the
    // terms and weights two further (a bound's address needs the term).  Eight waves each doing
    // this spent a sixth of the pass's vector instructions on it: 48.0 ms for 7,000 queries over
    // 8.8M documents, 46.4 from one planner; 19.0 and 17.8 ms with alpha 0.2, beta 0.8, where a
    // tile has fewer chunks.  The last wave plans: short queries leave it without chunks.
    __shared__ Lists s_lists[kWave];
    const bool planner = wave == NW - 1;
    int32_t term2 = 0;
    float w1 = 0.0f, w2 = 0.0f;
    uint32_t lo = 0, hi = 0;  // lanes past the query's terms read term 0's bounds and ignore them
    auto ahead = [&](int32_t i) {  // bounds of query i, whose terms are loaded, and terms of i + 1
        lo = toff[term2];
        hi = toff[term2 + 1];
        w1 = w2;
        terms(i + 1, term2, w2);
    };
    if (planner) {
        terms(0, term2, w2);
        ahead(0);
        s_lists[lane] = plan(lo, hi, lane < (__builtin_amdgcn_readlane(r_n, 0) & 0xFFFF), w1);
        ahead(1);
    }
    __syncthreads();

    for (int32_t i = 0; i < m; ++i) {
        const int32_t slot = s0 + i;
        const int32_t ni = __builtin_amdgcn_readlane(r_n, i);
        const int32_t n = ni & 0xFFFF, nseg = (n + kWave - 1) / kWave;
        const bool imp = (ni & (1 << 16)) != 0;
        if (i == m - 1) last();
        for (int32_t s = 0; s < nseg; ++s) {
            Lists ls;
            if (s == 0) {
                ls = s_lists[lane];
            } else {  // lane l holds list 64 s + l
                const int64_t qa = readlane64(r_qa, i);
                const int32_t li = s * kWave + lane;
                int32_t term = 0;
                float w = 0.0f;
                if (li < n) {
                    term = (ct + qa)[li];
                    w = (cw + qa)[li];
                }
                ls = plan(toff[term], toff[term + 1], li < n, w);
            }
            const uint32_t st = (uint32_t)__builtin_amdgcn_readlane((int)ls.cpn, kWave - 1);
            if (st == 0) continue;
            // list of chunk ci: the lanes whose lists end at or before ci, counted
            const uint32_t cpn = ls.cpn, basel = ls.basel, endl = ls.endl;
            const float wl = ls.w;
            auto take = [&]() {  // the first chunk of the wave's next batch
                uint32_t g = 0;
                if (lane == 0) g = atomicAdd(&s_next[s], (uint32_t)KU);
                return uni(g);
            };
            const uint32_t lb = st;
            uint32_t cs = (uint32_t)wave * (uint32_t)KU;
            // The list of the wave's last chunk: its chunks end at c_end, its chunk 0 would
            // start at group l_base, it ends at group l_end, its weight is l_w.  A wave's chunk
            // numbers only grow inside a segment, so a chunk below c_end is in that list.
            uint32_t c_end = 0, l_base = 0, l_end = 0;
            float l_w = 0.0f;
            while (cs < lb) {
                uint2 ids[KU];
                Raw raw[KU];
                uint32_t nl[KU];
                float wk[KU];
                // Loads are unconditional, so they leave back to back: lane l reads
                // group g0 + l even past its chunk's end (at most 63 groups past the
                // tile's last group: inside the arrays); those lanes add nothing.
                // The wave issues them at raised priority, so waves about to load
                // go ahead of waves adding into LDS.
                __builtin_amdgcn_s_setprio(3);
#pragma unroll
                for (int i = 0; i < KU; ++i) {
                    const uint32_t ci = cs + (uint32_t)i;
                    uint32_t g0 = 0, nn = 0;
                    if (ci < lb) {  // wave-uniform
                        if (ci >= c_end) {  // the next list holding chunks
                            const int k = (int)__popcll(__ballot(cpn <= ci));
                            c_end = (uint32_t)__builtin_amdgcn_readlane((int)cpn, k);
                            l_base = (uint32_t)__builtin_amdgcn_readlane((int)basel, k);
                            l_end = (uint32_t)__builtin_amdgcn_readlane((int)endl, k);
                            l_w = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wl), k));
                        }
                        g0 = l_base + ci * (uint32_t)kChunk;
                        nn = min((uint32_t)kChunk, l_end - g0);
                        g0 = min(g0, n_groups);
                    }
                    wk[i] = l_w;
                    nl[i] = nn;
                    const uint32_t gi = g0 + (uint32_t)lane;
                    load_at(pd_t, gi * (uint32_t)sizeof(uint2), ids[i]);
                    load_at(pv_t, gi * (uint32_t)sizeof(Raw), raw[i]);
                }
                __builtin_amdgcn_s_setprio(0);
                const uint32_t next = take();  // while this batch's loads are in flight
#pragma unroll
                for (int i = 0; i < KU; ++i) {
                    if ((uint32_t)lane >= nl[i]) continue;
                    const float w = wk[i];
                    // byte offsets of the documents' 32-bit score words
                    const uint32_t d4[4] = {ids[i].x & 0xFFFFu, ids[i].x >> 16, ids[i].y & 0xFFFFu,
                                            ids[i].y >> 16};
#pragma unroll
                    for (int p = 0; p < 4; ++p)
                        lds_add_i32(reinterpret_cast<int32_t *>(smem + d4[p]),
                                    (int32_t)Val<VT>::prod(raw[i], p, w));
                }
                // Every slot's loads are complete here, also those of slots that
                // added nothing: no load of this batch is then still in flight when
                // the next batch (or the next tile's first, behind the list-bounds
                // prefetch) reuses its registers, so those loads never wait.
#pragma unroll
                for (int i = 0; i < KU; ++i) __asm__ volatile("" ::"v"(ids[i].x), "v"(raw[i].x));
                cs = next;
            }
        }
        Lists next;
        const bool plans = planner && i + 1 < m;
        if (plans) next = plan(lo, hi, lane < (__builtin_amdgcn_readlane(r_n, i + 1) & 0xFFFF), w1);
        __syncthreads();
        if (plans) {
            s_lists[lane] = next;
            ahead(i + 2);
        }
        if (tid < nseg) s_next[tid] = kFirstTaken;  // every wave has taken its last batch

        // ---- read the row: sample maxima or emit every score at or above the
        // query's threshold (as in k_accumulate; a threshold that no sum reaches is INT32_MAX,
        // and sums stay within 2^30)
        const float qinv = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(r_qinv), i));
        const int32_t th = __builtin_amdgcn_readlane(r_th, i);
        if (SAMPLE) {
            int32_t mx = INT32_MIN;
            int m = tid;
            for (; m + 7 * NT < len; m += 8 * NT) {  // eight in flight
                int32_t v[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) v[k] = lds_take(A32 + m + k * NT);
#pragma unroll
                for (int k = 0; k < 8; ++k) mx = max(mx, v[k]);
            }
            for (; m < len; m += NT) mx = max(mx, lds_take(A32 + m));
            const acc_args_t h = acc_args();
            h->maxima[((size_t)slot * h->n_sample + ti) * NT + tid] = tid < len ? (float)mx * qinv : -INFINITY;
        } else {
            // The wave's steps: 256 sums each, NW * 256 apart, cleared as they are read.
            const int4 zero = fresh_zero4();  // one per read-out: the loops keep it live
            int base = wave * 256;
            if (!every && !imp) {
                // The sums of K steps that reach the threshold.  Few lanes with any (the common
                // case): each takes its own place in the workgroup's buffer.  Many lanes, or no room:
                // the sums go back to the row, then one place in the buffer for all of the wave's and,
                // for what lies past its end, one in the list.  (Atomics on one word take 12 ns each,
                // and a query whose pool comes from few tiles has hundreds of candidates in each.
                // With an atomic for each past the buffer's end, 1,000 queries over 40,000 documents,
                // gamma 1,000, took 2.85 ms, 0.41 so; over 100,000, gamma 4,096, 36.1 and 2.2; 300,000
                // in topical order, gamma 500, 0.89 and 0.70.  Without the first case 8.8M documents
                // with alpha 0.2, beta 0.8 take 4% longer; its limit may be 1 to 16.)
                auto place = [&](const auto &r, int m0) {
                    constexpr int K = sizeof(r) / sizeof(int4);
                    int32_t mx[K], most = INT32_MIN;
#pragma unroll
                    for (int k = 0; k < K; ++k) {
                        mx[k] = max(max(r[k].x, r[k].y), max(r[k].z, r[k].w));
                        most = max(most, mx[k]);
                    }
                    const int32_t lanes = (int32_t)__popcll(__ballot(most >= th));
                    if (lanes == 0) return;
                    const bool few = lanes <= kFewHits;
                    uint32_t todo = 0;  // bit e: the sum at document at(e) is still to be placed
                    auto at = [&](int e) { return m0 + (e >> 2) * NW * 256 + (e & 3); };
                    auto hit = [&](int32_t v, int e) {
                        if (v < th) return;
                        if (few) {
                            const uint32_t j = atomicAdd(&s_cand_n, 1u);
                            if (j < kCandBuf) {
                                s_cand[j] = ((uint64_t)(uint32_t)v << 32) | (uint32_t)(i << 16 | at(e));
                                return;
                            }
                        }
                        A32[at(e)] = v;
                        todo |= 1u << e;
                    };
#pragma unroll
                    for (int k = 0; k < K; ++k) {
                        if (mx[k] < th) continue;
                        hit(r[k].x, 4 * k);
                        hit(r[k].y, 4 * k + 1);
                        hit(r[k].z, 4 * k + 2);
                        hit(r[k].w, 4 * k + 3);
                    }
                    if (__ballot(todo != 0) == 0) return;
                    const uint32_t mine = (uint32_t)__popc(todo), incl = wave_incl_scan(mine);
                    const uint32_t n = (uint32_t)__builtin_amdgcn_readlane((int)incl, kWave - 1);
                    uint32_t first = 0, pos = 0;
                    if (lane == 0) first = atomicAdd(&s_cand_n, n);
                    first = uni(first);
                    const acc_args_t h = acc_args();
                    if (first + n > kCandBuf) {
                        const uint32_t past = max(first, kCandBuf);  // the first number past the buffer
                        if (lane == 0) pos = atomicAdd(h->count + slot, first + n - past);
                        pos = uni(pos) - past;
                    }
                    for (uint32_t j = first + incl - mine; todo; todo &= todo - 1u, ++j) {
                        const int m = at(__ffs(todo) - 1);
                        const int32_t v = lds_take(A32 + m);
                        if (j < kCandBuf)
                            s_cand[j] = ((uint64_t)(uint32_t)v << 32) | (uint32_t)(i << 16 | m);
                        else if ((int64_t)(pos + j) < h->cap)
                            h->cand[(size_t)slot * h->cap + (pos + j)] =
                                make_key((float)v * qinv, (uint32_t)(d0 + m));
                    }
                };
                // whole steps, four of them read together (most hold no candidate), then at most
                // one across the tile's end.  Sums that are not there read INT32_MIN: the threshold
                // is above zero here, so they are no candidates.
                for (; base + 256 <= len; base += 4 * NW * 256) {
                    const int m0 = base + lane * 4;
                    int4 r[4];
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        r[k] = make_int4(INT32_MIN, INT32_MIN, INT32_MIN, INT32_MIN);
                        if (base + k * NW * 256 + 256 <= len) {  // uniform
                            r[k] = lds_take4(A32 + m0 + k * NW * 256);
                        }
                    }
                    place(r, m0);
                }
                base = wave * 256 + (len - wave * 256) / (NW * 256) * (NW * 256);
                if (wave * 256 < len && base + 256 > len) {  // uniform
                    const int m0 = base + lane * 4;
                    int4 r[1] = {make_int4(INT32_MIN, INT32_MIN, INT32_MIN, INT32_MIN)};
                    if (m0 < len) {
                        r[0] = *reinterpret_cast<const int4 *>(A32 + m0);
                        *reinterpret_cast<int4 *>(A32 + m0) = zero;
                        if (m0 + 1 >= len) r[0].y = INT32_MIN;
                        if (m0 + 2 >= len) r[0].z = INT32_MIN;
                        if (m0 + 3 >= len) r[0].w = INT32_MIN;
                    }
                    place(r, m0);
                }
            } else {
                const acc_args_t h = acc_args();
                uint64_t *list = h->cand + (size_t)slot * h->cap;
                for (; base < len; base += NW * 256) {
                    const int m0 = base + lane * 4;
                    int4 r = make_int4(0, 0, 0, 0);
                    if (m0 < len) {
                        r = *reinterpret_cast<const int4 *>(A32 + m0);
                        *reinterpret_cast<int4 *>(A32 + m0) = zero;
                    }
                    const float sv[4] = {(float)r.x * qinv, (float)r.y * qinv, (float)r.z * qinv,
                                         (float)r.w * qinv};
                    if (every) {  // no threshold: each document at its own place
#pragma unroll
                        for (int p = 0; p < 4; ++p)
                            if (m0 + p < len) list[d0 + m0 + p] = make_key(sv[p], (uint32_t)(d0 + m0 + p));
                        continue;
                    }
                    // threshold <= 0: every nonzero sum, negative ones included, so that the finalize
                    // kernel may take each document left out as a zero
                    const bool ok[4] = {r.x != 0 && m0 < len, r.y != 0 && m0 + 1 < len,
                                        r.z != 0 && m0 + 2 < len, r.w != 0 && m0 + 3 < len};
                    if (__ballot(ok[0] || ok[1] || ok[2] || ok[3]))
                        emit_candidates<4>(sv, ok, d0 + m0, h->count + slot, list, h->cap);
                }
            }
        }
        __syncthreads();
        if (!SAMPLE) {
            // Every wave reads the same count here: the next query's read-out, behind a barrier,
            // is the next to change it.
            const uint32_t held = min(uni(s_cand_n), kCandBuf);
            if (lane == i) r_end = held;
            if (held > kCandBuf / 2 || (i == m - 1 && held > 0)) {
                // one place in its candidate list for each query's entries, all queries at once
                const acc_args_t h = acc_args();
                if (wave == 0) {
                    const uint32_t below = (uint32_t)__shfl_up((int)r_end, 1, kWave);
                    const uint32_t start = lane == i_flush ? 0u : below;
                    if (lane >= i_flush && lane <= i && r_end > start)
                        s_place[lane] = atomicAdd(h->count + s0 + lane, r_end - start) - start;
                }
                __syncthreads();
                for (uint32_t e = tid; e < held; e += NT) {
                    const uint64_t x = s_cand[e];
                    const int32_t j = (int32_t)((uint32_t)x >> 16), local = (int32_t)(x & 0xFFFFu);
                    const float s = (float)(int32_t)(x >> 32) *
                                    h->c.qinv[h->slots.rows ? h->slots.rows[s0 + j] : h->slots.row0 + s0 + j];
                    const uint32_t pos = s_place[j] + e;
                    if ((int64_t)pos < h->cap)
                        h->cand[(size_t)(s0 + j) * h->cap + pos] = make_key(s, (uint32_t)(d0 + local));
                }
                i_flush = i + 1;
                if (tid == 0) s_cand_n = 0;
            }
        }
    }
}

// One workgroup per item: grid (items of a tile, tiles over two dimensions).
template <int VT, bool SAMPLE>
__global__ __launch_bounds__(kAccThreads) __attribute__((amdgpu_waves_per_eu(6))) void k_accumulate1(AccArgs)
{
    const acc_args_t g = acc_args();
    const int64_t ti = (int64_t)blockIdx.z * gridDim.y + blockIdx.y;
    if (ti >= g->items.tiles) return;  // the whole workgroup
    const int32_t s0 = (int32_t)blockIdx.x * g->items.run;
    accumulate1_item<VT, SAMPLE>(ti, s0, min(s0 + g->items.run, g->slots.n), true, [] {});
}

// The same work as one persistent launch fed by device work queues: as many workgroups as
// the device holds at once, each starting with the item of its own index and taking the next
// from its queue's counter until the items are used up (the counter is read as an item's last
// query starts, so the wait for it is hidden), then from the other queues'.  Items run in the
// grid's order, so the workgroups of a queue score the same tile, and a caller that orders its
// slots by decreasing work starts the long queries of each tile first.  Workgroups go to the
// eight XCDs in turn, so with eight queues a tile's lists are read by one XCD and stay in its L2;
// with one queue every L2 held the lists of the one to three tiles in work.  256 queries over 1M
// unpruned documents (16 MB a tile), scoring pass 1.54 -> 1.05 ms; 1,000 over 1M documents of 250K
// terms 0.50 -> 0.48, the sampling pass 0.107 -> 0.077.  Fewer than four items a workgroup stay in
// one queue (37 queries, 24 tiles: 30 us, 43 from eight): all workgroups come back at once there.
// A workgroup leaves once it has found every queue's counter past its last item; the counters
// (kQueueStep words apart) must be 0 at launch.
template <int VT, bool SAMPLE>
__global__ __launch_bounds__(kAccThreads) __attribute__((amdgpu_waves_per_eu(6))) void k_accumulate1_queue(AccArgs)
{
    __shared__ int64_t s_item;
    uint32_t x = blockIdx.x % (uint32_t)acc_args()->items.queues;  // the queue, and the item's place in it
    int64_t j = blockIdx.x / (uint32_t)acc_args()->items.queues;
    // The first wave: the next item as j * kQueues + x, from queue x on; -1: none is left.  Past the
    // end of its own queue it looks at all counters at once before it takes from another: at the
    // end of the launch every workgroup comes by, and atomics on one word take 12 ns each.
    auto take = [&]() -> int64_t {
        const acc_args_t h = acc_args();
        const uint32_t nq = (uint32_t)h->items.queues, y = threadIdx.x & (kWave - 1);
        const int64_t begin = (gridDim.x - y + nq - 1) / nq;  // lane y < nq: queue y
        const int64_t left = (int64_t)((h->items.tiles - y + nq - 1) / nq) * h->items.groups - begin;
        uint32_t from = x;
        for (;;) {
            int64_t i = 0;
            if (y == from) i = (int64_t)atomicAdd(h->head + y * kQueueStep, 1ull);
            if (__ballot(y == from && i < left)) {
                const uint64_t it = (uint64_t)((begin + i) * kQueues + y);
                return readlane64((int64_t)it, (int)from);
            }
            if (nq == 1) return -1;
            const uint64_t open = __ballot(
                y < nq && (int64_t)__hip_atomic_load(h->head + (y < nq ? y : 0) * kQueueStep, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT) < left);
            if (open == 0) return -1;
            const uint64_t on = open >> from << from;  // the next open one from there, in turn
            from = (uint32_t)__builtin_ctzll(on ? on : open);
        }
    };
    bool first = true;
    for (;;) {
        const acc_args_t g = acc_args();
        const int64_t row = j / g->items.groups;
        const int64_t ti = row * g->items.queues + x;
        int64_t next = -1;
        const int32_t s0 = (int32_t)(j - row * g->items.groups) * g->items.run;
        accumulate1_item<VT, SAMPLE>(ti, s0, min(s0 + g->items.run, g->slots.n), first, [&] {
            if (threadIdx.x < kWave && acc_args()->items.n > gridDim.x) next = take();
        });
        first = false;
        if (acc_args()->items.n <= gridDim.x) break;  // an item each (the host sets one queue)
        // (the item's own barriers lie between this write and the last read)
        if (threadIdx.x == 0) s_item = next;
        __syncthreads();
        const int64_t it = uni64(s_item);
        if (it < 0) break;
        x = (uint32_t)it % kQueues;
        j = it / kQueues;
    }
}

// ------------------------------------------------------------------ threshold
// theta = the rank-th largest sampled maximum.  Both accumulate passes
// produce bitwise identical scores (integer sums), so every sampled document
// at or above theta is kept again by the scoring pass.  The finalize kernel
// verifies the result (at least gamma candidates kept).
//
// Bound by the barriers of its select; a thread keeps up to R maxima in registers.  One query
// (4,096 maxima): 4.7 us; 7,000 queries: 40 us (7.8 and 150 us with four fixed digits from memory).
template <int NT, int R>
__global__ __launch_bounds__(NT) void k_theta(const float *maxima, int64_t n_m, int64_t rank,
                                              DevSlots slots, const float *qinv, float *theta,
                                              int32_t *sum_min)
{
    __shared__ SelectLds L;
    __shared__ uint32_t s_min;
    const float *mx = maxima + (size_t)blockIdx.x * (size_t)n_m;
    const int tid = threadIdx.x;
    if (tid == 0) s_min = 0xFFFFFFFFu;
    auto select = [&](auto each) {
        bool exact;
        const uint32_t t = block_select<NT, uint32_t>(ord_f32(mx[0]), rank, each, L, &exact);
        if (exact) return t;
        uint32_t mn = 0xFFFFFFFFu;  // the least key at or above the bound is the rank-th largest
        each([&](uint32_t k) { mn = k >= t ? min(mn, k) : mn; });
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) mn = min(mn, (uint32_t)__shfl_xor(mn, m, kWave));
        if ((tid & (kWave - 1)) == 0) atomicMin(&s_min, mn);
        __syncthreads();
        return s_min;
    };
    uint32_t key;
    if (n_m <= NT * R) {
        uint32_t k[R];
#pragma unroll
        for (int j = 0; j < R; ++j) k[j] = j * NT + tid < n_m ? ord_f32(mx[j * NT + tid]) : 0u;
        key = select([&](auto f) {
#pragma unroll
            for (int j = 0; j < R; ++j)
                if (j * NT + tid < n_m) f(k[j]);
        });
    } else {
        key = select([&](auto f) {
            for (int64_t i = tid; i < n_m; i += NT) f(ord_f32(mx[i]));
        });
    }
    if (tid >= kWave) return;
    float th = unord_f32(key);
    th = th > -INFINITY ? th : -INFINITY;
    // Fewer sampled maxima than the rank (tiles of fewer documents than threads): every document
    // would be kept, more than the candidate list holds (a threshold is only taken where the corpus
    // exceeds the list).  The scoring pass then emits none, and the row, short of its pool, is left to
    // the retry: 1,000 queries over 37,600 documents, gamma 815, 0.49 ms, 24.0 with every document
    // emitted one by one.
    const int32_t a = th > -INFINITY ? sum_threshold_wave(th, qinv[slots.row(blockIdx.x)]) : INT32_MAX;
    if (tid == 0) {
        theta[blockIdx.x] = th;
        sum_min[blockIdx.x] = a;
    }
}

__global__ void k_fill_f32(float *p, int64_t n, float v)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}
__global__ void k_fill_u32(uint32_t *p, int64_t n, uint32_t v)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}
// What the host reads when a pass has ended: the rows that need a retry, the query flags and the
// longest row, into pinned host memory.
__device__ __forceinline__ void write_report(const DevRetry &r)
{
    __hip_atomic_store(&r.report->left, *r.count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(&r.report->flags, (uint32_t)r.err[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(&r.report->longest, (uint32_t)r.err[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
// On its own: for a host that waits for the words and not for the stream.
__global__ void k_report(DevRetry r)
{
    write_report(r);
    __hip_atomic_store(&r.report->there, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// ------------------------------------------------------------------ finalize
// Leave a row to a retry pass (one thread, once per row).
__device__ __forceinline__ void retry_row(const DevRetry &r, int32_t row)
{
    r.status[row] = kSlotRetry;
    r.rows[atomicAdd(r.count, 1u)] = row;
}

// The full (unpruned) query row in LDS: 2^lg buckets of two entries {term, term, value, value},
// empty terms -1.  A term sits in its home bucket or, where that is full, in the next one with
// room; `spill` says whether any term did that.  With eight buckets per term few tables spill
// (n^3 / 6 B^2: 3% at 35 terms and 512 buckets), and a lookup is then one 16-byte LDS read and
// two compares with no loop: an open-addressing table of half the size ran its probe loop about
// three times per 64 lanes, which is what bounded the rerank (see k_rerank).
struct QueryTable {
    int4 *b;
    int32_t lg;
    uint32_t spill;
};
constexpr int kTableLgMax = 12;  // 64 KB; holds the longest row (kQueryHash / 2 terms)

__host__ __device__ __forceinline__ int table_lg(int64_t n)
{
    int lg = 6;
    while (lg < kTableLgMax && (1ll << lg) < 8 * n) ++lg;
    return lg;
}

// Byte offset of a term's home bucket (Fibonacci hashing of the term's low 24 bits).
__device__ __forceinline__ uint32_t home_bucket(int32_t id, int lg)
{
    return (__umul24((uint32_t)id, 0x9E3779u) >> (20 - lg)) & (((1u << lg) - 1u) << 4);
}

// Fill the table from the query row [a, b): every thread of the workgroup, two barriers.
// s_spill: a word of LDS.  With POS the buckets hold the terms' positions in the row instead of
// their values.
template <bool POS>
__device__ __forceinline__ void build_table(const DevQueries &q, int64_t a, int64_t b,
                                            QueryTable &t, uint32_t *s_spill)
{
    const int B = 1 << t.lg;
    for (int i = threadIdx.x; i < B; i += blockDim.x) t.b[i] = make_int4(-1, -1, 0, 0);
    if (threadIdx.x == 0) *s_spill = 0u;
    __syncthreads();
    for (int64_t e = a + threadIdx.x; e < b; e += blockDim.x) {
        const int32_t id = q.indices[e];
        const int32_t v = POS ? (int32_t)(e - a) : __float_as_int(q.values[e]);
        const uint32_t home = home_bucket(id, t.lg) >> 4;
        for (uint32_t i = home;; i = (i + 1) & (uint32_t)(B - 1)) {
            int32_t *k = reinterpret_cast<int32_t *>(t.b + i);
            const int s = atomicCAS(k, -1, id) == -1 ? 0 : (atomicCAS(k + 1, -1, id) == -1 ? 1 : 2);
            if (s < 2) {
                k[2 + s] = v;
                if (i != home) *s_spill = 1u;
                break;
            }
        }
    }
    __syncthreads();
    t.spill = uni(*s_spill);
}

// The query's value of a term; false where it has none.  id -2 is no term.
__device__ __forceinline__ bool table_get(const QueryTable &t, int32_t id, float &v)
{
    uint32_t off = home_bucket(id, t.lg);
    int4 k = *reinterpret_cast<const int4 *>(reinterpret_cast<const unsigned char *>(t.b) + off);
    if (t.spill) {  // uniform: some term of this query is not in its home bucket
        while (k.x != id && k.y != id && k.y != -1) {
            off = (off + 16) & (((1u << t.lg) - 1u) << 4);
            k = *reinterpret_cast<const int4 *>(reinterpret_cast<const unsigned char *>(t.b) + off);
        }
    }
    v = __int_as_float(k.x == id ? k.z : k.w);
    return k.x == id || k.y == id;
}

// The wave-wide sums of four values at once, each in the pairing of a butterfly over lane
// distances 32, 16, 8, 4, 2, 1: lane l gets the sum of value (l >> 5) + 2 ((l >> 4) & 1).  The
// halves and rows of two values are swapped into one register, so a stage adds two values' halves
// with one instruction.
__device__ __forceinline__ float wave_sum4(float a, float b, float c, float d)
{
    auto swap32 = [](float x, float y) {
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
        return __uint_as_float(r[0]) + __uint_as_float(r[1]);
    };
    auto swap16 = [](float x, float y) {
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
        return __uint_as_float(r[0]) + __uint_as_float(r[1]);
    };
    float s = swap16(swap32(a, b), swap32(c, d));
    // rotations within rows of 16 lanes: after the stage at distance d the values repeat every d
    // lanes, so a rotation by d / 2 reads the partner
    s += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(s), 0x128, 0xF, 0xF, false));
    s += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(s), 0x124, 0xF, 0xF, false));
    s += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(s), 0x122, 0xF, 0xF, false));
    s += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(s), 0x121, 0xF, 0xF, false));
    return s;
}

// The bounds (uniform) and the first two 64-entry rounds of four corpus rows, all loads in
// flight together; lanes past a row's end hold term -2.
struct Rows4 {
    int64_t at[4];
    int32_t n[4];
    int32_t id[4][2];
    float x[4][2];
    __device__ __forceinline__ void load(const DevIndex &ix, const int64_t (&ra)[4],
                                         const int64_t (&rb)[4])
    {
        const int lane = threadIdx.x & (kWave - 1);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            at[j] = uni64(ra[j]);
            n[j] = (int32_t)uni((uint32_t)(rb[j] - ra[j]));
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                id[j][r] = -2;
                x[j][r] = 0.0f;
                if (r * kWave + lane < n[j]) {
                    id[j][r] = (ix.indices + at[j])[r * kWave + lane];
                    x[j][r] = (ix.values + at[j])[r * kWave + lane];
                }
            }
        }
    }
    // delta(q, x_j) in FP32 of the four rows: each lane over entries lane, lane + 64, ... of the
    // row in order, then summed across the wave (as wave_sum4 leaves them)
    __device__ __forceinline__ float dot(const DevIndex &ix, const QueryTable &tb) const
    {
        const int lane = threadIdx.x & (kWave - 1);
        float acc[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            acc[j] = 0.0f;
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                float v;
                if (table_get(tb, id[j][r], v)) acc[j] = fmaf(v, x[j][r], acc[j]);
            }
            for (int32_t p = 2 * kWave + lane; p < n[j]; p += kWave) {
                float v;
                if (table_get(tb, (ix.indices + at[j])[p], v))
                    acc[j] = fmaf(v, (ix.values + at[j])[p], acc[j]);
            }
        }
        return wave_sum4(acc[0], acc[1], acc[2], acc[3]);
    }
};
// The row whose sum wave_sum4 leaves in this lane.
__device__ __forceinline__ int sum4_row()
{
    const int lane = threadIdx.x & (kWave - 1);
    return (lane >> 5) + 2 * ((lane >> 4) & 1);
}

// LDS sizes: P = the power of two at or above need keys, a rerank table of
// 2^tlg buckets, tlg = table_lg of the longest query row of the launch.
__host__ __device__ inline int32_t pow2_at_least(int32_t n)
{
    int32_t p = 1;
    while (p < n) p <<= 1;
    return p;
}

// The m keys (distinct) in LDS, descending, as (id, score) into the first k places of the query's
// output row, padded with (-1, -inf).  Up to kRankSort keys each find their place by counting the
// larger ones, with no further barrier; more are sorted (bitonic; keys has pow2_at_least(m) words).
template <int NT>
__device__ void sort_and_write(uint64_t *keys, int32_t m, int32_t k, int32_t row,
                               int64_t *out_ids, float *out_scores)
{
    const int tid = threadIdx.x;
    int64_t *ids = out_ids + (size_t)row * (size_t)k;
    float *sc = out_scores + (size_t)row * (size_t)k;
    for (int r = m + tid; r < k; r += NT) {
        ids[r] = -1;
        sc[r] = -INFINITY;
    }
    if (m <= kRankSort) {
        __syncthreads();
        for (int i = tid; i < m; i += NT) {
            const uint64_t key = keys[i];
            int32_t rank = 0;
#pragma unroll 4
            for (int j = 0; j < m; ++j) rank += keys[j] > key ? 1 : 0;
            if (rank < k) {
                ids[rank] = (int64_t)key_doc(key);
                sc[rank] = key_score(key);
            }
        }
        return;
    }
    const int32_t P = pow2_at_least(m);
    for (int i = m + tid; i < P; i += NT) keys[i] = 0ull;
    __syncthreads();
    for (int kk = 2; kk <= P; kk <<= 1) {
        for (int j = kk >> 1; j > 0; j >>= 1) {
            for (int i = tid; i < P; i += NT) {
                const int ij = i ^ j;
                if (ij > i) {
                    const uint64_t x = keys[i], y = keys[ij];
                    const bool desc = (i & kk) == 0;
                    if (desc ? (x < y) : (x > y)) {
                        keys[i] = y;
                        keys[ij] = x;
                    }
                }
            }
            __syncthreads();
        }
    }
    for (int r = tid; r < min(m, k); r += NT) {
        ids[r] = (int64_t)key_doc(keys[r]);
        sc[r] = key_score(keys[r]);
    }
}

// The next place in an LDS list for every lane with `take`: one atomic per wave.
__device__ __forceinline__ uint32_t wave_place(uint32_t *n, bool take)
{
    const uint64_t m = __ballot(take);
    uint32_t base = 0;
    if (m == 0) return 0;
    const int first = __ffsll((unsigned long long)m) - 1;
    if ((int)(threadIdx.x & (kWave - 1)) == first) base = atomicAdd(n, (uint32_t)__popcll(m));
    return (uint32_t)__builtin_amdgcn_readlane((int)base, first) + lanes_below(m);
}

// One workgroup per query slot: the exact top-need of its coarse candidates
// (with the zero-score documents the scoring pass left implicit).  Without a
// rerank it sorts them and writes the top k; with a rerank it writes them to
// pool[slot][need] for k_rerank and k_topk.
//
// Bound by latency: the candidates' load and the barriers of the select.  Up to NT R candidates
// stay in registers over its passes.  One query (about 1,500 candidates): 5.9 us; 10,000
// candidates (every document of a small index) 8.3 us; 7,000 queries 45 us (14.8, 60 and 124 us
// with eight fixed digits from memory).
template <bool RERANK, int NT, int R>
__global__ __launch_bounds__(NT) void k_finalize(
    DevIndex ix, DevSlots slots, const uint32_t *count, const uint64_t *cand,
    const float *theta, int64_t cap, int32_t need, int32_t k, int32_t bm_words, uint64_t *pool,
    int64_t *out_ids, float *out_scores, DevRetry retry)
{
    constexpr int NW = NT / kWave;
    extern __shared__ __align__(16) unsigned char smem[];
    const int32_t P = pow2_at_least(need);
    uint64_t *keys = reinterpret_cast<uint64_t *>(smem);                   // [P]
    // the bitmap of the implicit zeros and the select's tables, used in turn
    uint32_t *bm = reinterpret_cast<uint32_t *>(keys + P);                  // [bm_words]
    SelectLds &L = *reinterpret_cast<SelectLds *>(keys + P);
    __shared__ uint32_t s_n, s_wsum[NW];
    const int tid = threadIdx.x;
    const int32_t slot = blockIdx.x;
    if (retry.unchecked && retry.err[0]) return;  // malformed queries: no output is written
    const int32_t row = slots.row(slot);
    // without a threshold every document is a candidate, at its own place
    const uint32_t cnt = theta ? count[slot] : (uint32_t)ix.n_docs;
    const float th = theta ? theta[slot] : -INFINITY;
    // threshold <= 0: the scoring pass emitted only nonzero sums; every document it did
    // not emit scores exactly 0
    const bool imp = th <= 0.0f && th != -INFINITY;
    if ((int64_t)cnt > cap || (!imp && (int64_t)cnt < (int64_t)need)) {
        if (tid == 0) retry_row(retry, row);
        return;
    }
    const uint64_t *cs = cand + (size_t)slot * (size_t)cap;
    constexpr uint32_t kZeroOrd = 0x80000000u;  // ord_f32(0.0f)
    if (tid == 0) s_n = 0;
    // the pool into keys; false: the slot needs a retry.  each(f): f on every candidate of the thread
    auto select = [&](auto each) -> bool {
        uint32_t n_pos = cnt;
        if (imp) {
            uint32_t mine = 0;
            each([&](uint64_t key) { mine += (uint32_t)(key >> 32) > kZeroOrd ? 1u : 0u; });
            (void)block_excl_scan<NT>(mine, s_wsum, n_pos);
        }
        if (!imp || (int64_t)n_pos >= (int64_t)need) {
            // the first need candidates (all positive when zeros are implicit)
            const uint64_t bound = (int64_t)cnt == need ? 0ull
                : block_select<NT, uint64_t>(cs[0], need, each, L, nullptr);
            __syncthreads();
            each([&](uint64_t key) {
                const bool take = key >= bound;
                const uint32_t p = wave_place(&s_n, take);
                if (take && p < (uint32_t)P) keys[p] = key;
            });
            __syncthreads();
            return true;
        }
        // every positive candidate, then the lowest-id zero-score documents, then (only if
        // the zeros run out) the best emitted negatives
        const int64_t zeros_avail = ix.n_docs - (int64_t)cnt;
        const int64_t zt = min((int64_t)need - n_pos, zeros_avail);
        const int64_t nt = (int64_t)need - n_pos - zt;
        const int64_t bound = min(ix.n_docs, zt + (int64_t)cnt);  // the zt-th zero id is below
        const int32_t words = (int32_t)((bound + 31) / 32);
        if (nt > (int64_t)cnt - n_pos || words > bm_words) return false;
        __syncthreads();
        each([&](uint64_t key) {
            const bool take = (uint32_t)(key >> 32) > kZeroOrd;
            const uint32_t p = wave_place(&s_n, take);
            if (take) keys[p] = key;
        });
        for (int w = tid; w < words; w += NT) bm[w] = 0u;
        __syncthreads();
        each([&](uint64_t key) {
            const uint32_t d = key_doc(key);
            if ((int64_t)d < bound) atomicOr(&bm[d >> 5], 1u << (d & 31));
        });
        __syncthreads();
        // zero bits in order: each thread owns a run of words
        const int32_t per = (words + NT - 1) / NT;
        const int32_t w0 = min(words, tid * per), w1 = min(words, w0 + per);
        auto free_bits = [&](int32_t w) {
            uint32_t m = ~bm[w];
            const int64_t top = bound - (int64_t)w * 32;  // valid bits in this word
            if (top < 32) m &= (1u << top) - 1u;
            return m;
        };
        uint32_t mine = 0;
        for (int32_t w = w0; w < w1; ++w) mine += (uint32_t)__popc(free_bits(w));
        uint32_t tot;
        uint32_t rank = block_excl_scan<NT>(mine, s_wsum, tot);
        for (int32_t w = w0; w < w1 && (int64_t)rank < zt; ++w) {
            uint32_t m = free_bits(w);
            while (m && (int64_t)rank < zt) {
                const int b = __ffs(m) - 1;
                m &= m - 1u;
                keys[n_pos + rank] = make_key(0.0f, (uint32_t)(w * 32 + b));
                ++rank;
            }
        }
        if (nt > 0) {
            // the nt best negatives: non-negative keys map to 0 and rank below them
            auto neg = [&](auto f) {
                each([&](uint64_t key) { f((uint32_t)(key >> 32) < kZeroOrd ? key : 0ull); });
            };
            const uint64_t first = (uint32_t)(cs[0] >> 32) < kZeroOrd ? cs[0] : 0ull;
            __syncthreads();  // the bitmap gives way to the tables
            const uint64_t kthn = block_select<NT, uint64_t>(first, nt, neg, L, nullptr);
            if (tid == 0) s_n = 0;
            __syncthreads();
            neg([&](uint64_t key) {
                const bool take = key && key >= kthn;
                const uint32_t p = wave_place(&s_n, take);
                if (take) keys[n_pos + zt + p] = key;
            });
        }
        __syncthreads();
        return true;
    };
    bool ok;
    if (cnt <= (uint32_t)(NT * R)) {
        uint64_t key[R];
#pragma unroll
        for (int j = 0; j < R; ++j) key[j] = (uint32_t)(j * NT + tid) < cnt ? cs[j * NT + tid] : 0ull;
        ok = select([&](auto f) {
#pragma unroll
            for (int j = 0; j < R; ++j)
                if ((uint32_t)(j * NT + tid) < cnt) f(key[j]);
        });
    } else {
        ok = select([&](auto f) {
            for (int64_t i = tid; i < cnt; i += NT) f(cs[i]);
        });
    }
    if (tid == 0) {
        if (ok)
            retry.status[row] = kSlotOk;
        else
            retry_row(retry, row);
    }
    if (!ok) return;
    if (RERANK) {
        for (int i = tid; i < need; i += NT) pool[(size_t)slot * (size_t)need + i] = keys[i];
        return;
    }
    sort_and_write<NT>(keys, need, k, row, out_ids, out_scores);
}

// Exact rerank (Alg. 4): each wave scores kRerankPerWave pool entries at a
// time, `groups` times, NW waves per workgroup, grid (slot, entry block);
// each workgroup builds the query's table in LDS (2^tlg buckets) once for its
// groups x NW x kRerankPerWave entries.  The entry's key becomes (FP32
// inner product of the unpruned row with the full query, then inverted id).
// Slots not finalized are skipped.
//
// Bound by HBM where the queries are many: 7,000 queries' 500 rows of ~125 entries (3.5 GB) take
// 0.56 ms, 6.3 TB/s; with an open-addressing table probed in a loop, butterfly sums and vector row
// addresses the instructions bound it (1.37 ms).  A call of few queries is bound by the chain of
// key, row bounds and row loads, so it takes one group per wave: one query 8.3 us, 41 us with four
// groups on eight workgroups.
__global__ __launch_bounds__(kFinThreads) void k_rerank(DevIndex ix, DevQueries q,
                                                        DevSlots slots, int32_t need,
                                                        int32_t tlg, int32_t groups, uint64_t *pool,
                                                        DevRetry retry)
{
    constexpr int NW = kFinThreads / kWave, EPW = kRerankPerWave;
    static_assert(EPW == 4, "Rows4");
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ uint32_t s_spill;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = (int)uni((uint32_t)threadIdx.x / kWave);
    const int32_t slot = blockIdx.x;
    const int32_t row = slots.row(slot);
    // (with malformed queries the row bounds mean nothing and the statuses were not written)
    if ((retry.unchecked && retry.err[0]) || retry.status[row] != kSlotOk) return;
    const int64_t qa = q.indptr[row], qb = q.indptr[row + 1];
    QueryTable tb{reinterpret_cast<int4 *>(smem), table_lg(qb - qa), 0u};
    if (tb.lg > tlg) {  // the launch was sized for shorter rows
        if (threadIdx.x == 0 && blockIdx.y == 0) retry_row(retry, row);
        return;
    }
    uint64_t *e = pool + (size_t)slot * (size_t)need;
    uint32_t lo[EPW];
    int64_t ra[EPW], rb[EPW];
    // keys and row bounds of the wave's entries [c0, c0 + EPW)
    auto bounds = [&](int32_t c0) {
#pragma unroll
        for (int j = 0; j < EPW; ++j) {
            lo[j] = 0;
            ra[j] = rb[j] = 0;
            if (c0 + j < need) {
                const uint64_t key = e[c0 + j];
                lo[j] = (uint32_t)key;
                const uint32_t doc = key_doc(key);
                ra[j] = ix.indptr[doc];
                rb[j] = ix.indptr[doc + 1];
            }
        }
    };
    // The first group's keys and row bounds are loaded before the query table is
    // built, and the first two 64-entry rounds of every row of a group are loaded
    // together, so the entries' memory latencies overlap.
    const int32_t first = (int32_t)blockIdx.y * groups * NW;
    bounds((first + wave) * EPW);
    build_table<false>(q, qa, qb, tb, &s_spill);
    for (int g = 0; g < groups; ++g) {
        const int32_t c0 = (first + g * NW + wave) * EPW;
        if (c0 >= need) break;  // wave-uniform; no barrier follows
        Rows4 rows;
        rows.load(ix, ra, rb);
        const uint32_t l0 = lo[0], l1 = lo[1], l2 = lo[2], l3 = lo[3];
        // the next group's keys and bounds arrive while this one's rows are looked up
        if (g + 1 < groups) bounds(c0 + NW * EPW);
        const float sc = rows.dot(ix, tb);
        const int j = sum4_row();
        const uint32_t l = j == 0 ? l0 : (j == 1 ? l1 : (j == 2 ? l2 : l3));
        if ((lane & 15) == 0 && c0 + j < need) e[c0 + j] = ((uint64_t)ord_f32(sc) << 32) | l;
    }
}

// One workgroup per slot: the top k of the reranked pool, in order.  A short result (k up to
// kRankSort of a pool of up to kTopkRegs per thread) is selected first, so that only k keys are
// put in order: one query (50 of 500) 5.0 us, 7,000 queries 21 us where sorting the
// pool (a barrier for each of 45 exchange steps) took 18.4 and 96 us.
template <bool SELECT>
__global__ __launch_bounds__(kFinThreads) void k_topk(DevSlots slots, int32_t need, int32_t k,
                                                      const uint64_t *pool, int64_t *out_ids,
                                                      float *out_scores, DevRetry retry)
{
    constexpr int NT = kFinThreads;
    extern __shared__ __align__(16) unsigned char smem[];
    uint64_t *keys = reinterpret_cast<uint64_t *>(smem);  // [pow2_at_least(SELECT ? k : need)]
    const int tid = threadIdx.x;
    const int32_t slot = blockIdx.x;
    const int32_t row = slots.row(slot);
    if (slot == 0 && tid == 0) write_report(retry);  // the pass's last kernel
    if (retry.unchecked && retry.err[0]) return;
    const uint64_t *e = pool + (size_t)slot * (size_t)need;
    if constexpr (SELECT) {
        __shared__ SelectLds L;
        __shared__ uint32_t s_n;
        uint64_t key[kTopkRegs];
#pragma unroll
        for (int j = 0; j < kTopkRegs; ++j) key[j] = j * NT + tid < need ? e[j * NT + tid] : 0ull;
        const uint64_t any = e[0];
        if (retry.status[row] != kSlotOk) return;
        if (tid == 0) s_n = 0;
        auto each = [&](auto f) {
#pragma unroll
            for (int j = 0; j < kTopkRegs; ++j)
                if (j * NT + tid < need) f(key[j]);
        };
        const uint64_t bound = block_select<NT, uint64_t>(any, k, each, L, nullptr);
        each([&](uint64_t x) {
            const bool take = x >= bound;
            const uint32_t p = wave_place(&s_n, take);
            if (take && p < (uint32_t)k) keys[p] = x;  // keys are distinct: exactly k
        });
        sort_and_write<NT>(keys, k, k, row, out_ids, out_scores);
    } else {
        if (retry.status[row] != kSlotOk) return;
        for (int i = tid; i < need; i += NT) keys[i] = e[i];
        sort_and_write<NT>(keys, need, k, row, out_ids, out_scores);
    }
}

// ------------------------------------------------------------------ pair scores
// Row bounds of the candidates [c0, c0 + 4) of query b; ids outside the corpus give empty rows.
__device__ __forceinline__ void cand_bounds(const DevIndex &ix, const int64_t *cand, int64_t n_cand,
                                            int64_t b, int64_t c0, int64_t (&ra)[4], int64_t (&rb)[4])
{
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        ra[j] = rb[j] = 0;
        if (c0 + j < n_cand) {
            const int64_t d = cand[b * n_cand + c0 + j];
            if (d >= 0 && d < ix.n_docs) {
                ra[j] = ix.indptr[d];
                rb[j] = ix.indptr[d + 1];
            }
        }
    }
}

// Scores of listed pairs: grid (query, candidate block), four candidates per wave at a time,
// `groups` times, as k_rerank does.  Bound by the chain of id, row bounds and row loads, so the
// candidates of a query are split over workgroups until the chip is full: 256 queries x 100
// candidates of ~180 entries take 11 us (145 us with one workgroup per query).
__global__ __launch_bounds__(kFinThreads) void k_score_forward(DevIndex ix, DevQueries q,
                                                               const int64_t *cand, int32_t n_cand,
                                                               int32_t tlg, int32_t groups, float *out)
{
    constexpr int NW = kFinThreads / kWave;
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ uint32_t s_spill;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = (int)uni((uint32_t)threadIdx.x / kWave);
    const int64_t b = blockIdx.x;
    QueryTable tb{reinterpret_cast<int4 *>(smem), tlg, 0u};
    const int64_t first = (int64_t)blockIdx.y * groups * NW;
    int64_t ra[4], rb[4];
    cand_bounds(ix, cand, n_cand, b, (first + wave) * 4, ra, rb);
    build_table<false>(q, q.indptr[b], q.indptr[b + 1], tb, &s_spill);
    for (int32_t g = 0; g < groups; ++g) {
        const int64_t c0 = (first + (int64_t)g * NW + wave) * 4;
        if (c0 >= n_cand) break;  // wave-uniform; no barrier follows
        Rows4 rows;
        rows.load(ix, ra, rb);
        if (g + 1 < groups) cand_bounds(ix, cand, n_cand, b, c0 + NW * 4, ra, rb);
        const float s = rows.dot(ix, tb);
        const int j = sum4_row();
        if ((lane & 15) == 0 && c0 + j < n_cand) out[b * n_cand + c0 + j] = s;
    }
}

// Gradients of s[b][c] = delta(q_b, x_c): every common dimension t adds
// G[b][c] * x_c[t] to the query entry and G[b][c] * q_b[t] to the document
// entry.  Grid and row loads as in k_score_forward.  A workgroup sums its candidates' query side
// in LDS and adds it to the query's gradient; queries' workgroups and document entries shared by
// several queries meet in global atomics.  256 x 100 candidates: 28 us (164 us with one workgroup
// per query).
__global__ __launch_bounds__(kFinThreads) void k_score_backward(
    DevIndex ix, DevQueries q, const int64_t *cand, int32_t n_cand, int32_t tlg, int32_t groups,
    const float *grad, float *gq, float *gx)
{
    constexpr int NW = kFinThreads / kWave;
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ uint32_t s_spill;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = (int)uni((uint32_t)threadIdx.x / kWave);
    const int64_t b = blockIdx.x;
    const int64_t qa = q.indptr[b], qb = q.indptr[b + 1];
    const int n = (int)(qb - qa);
    QueryTable tb{reinterpret_cast<int4 *>(smem), tlg, 0u};
    float *qv = reinterpret_cast<float *>(tb.b + (1 << tlg));  // [n] the query's values
    float *gacc = qv + n;                                      // [n] its gradient's sums
    uint32_t *gtouch = reinterpret_cast<uint32_t *>(gacc + n); // [n] entries that got any
    const int64_t first = (int64_t)blockIdx.y * groups * NW;
    int64_t ra[4], rb[4];
    cand_bounds(ix, cand, n_cand, b, (first + wave) * 4, ra, rb);
    for (int i = threadIdx.x; i < n; i += kFinThreads) {
        qv[i] = q.values[qa + i];
        gacc[i] = 0.0f;
        gtouch[i] = 0u;
    }
    build_table<true>(q, qa, qb, tb, &s_spill);
    for (int32_t g = 0; g < groups; ++g) {
        const int64_t c0 = (first + (int64_t)g * NW + wave) * 4;
        if (c0 >= n_cand) break;  // wave-uniform
        Rows4 rows;
        rows.load(ix, ra, rb);
        float gr[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) gr[j] = c0 + j < n_cand ? grad[b * n_cand + c0 + j] : 0.0f;
        if (g + 1 < groups) cand_bounds(ix, cand, n_cand, b, c0 + NW * 4, ra, rb);
        auto entry = [&](int j, int32_t id, float x, int32_t p) {
            float at;
            if (!table_get(tb, id, at)) return;
            const int i = __float_as_int(at);
            if (gq) {
                lds_add(&gacc[i], gr[j] * x);
                gtouch[i] = 1u;
            }
            if (gx) atomicAdd(&gx[rows.at[j] + p], gr[j] * qv[i]);
        };
#pragma unroll
        for (int j = 0; j < 4; ++j) {
#pragma unroll
            for (int r = 0; r < 2; ++r) entry(j, rows.id[j][r], rows.x[j][r], r * kWave + lane);
            for (int32_t p = 2 * kWave + lane; p < rows.n[j]; p += kWave)
                entry(j, (ix.indices + rows.at[j])[p], (ix.values + rows.at[j])[p], p);
        }
    }
    if (!gq) return;
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += kFinThreads)
        if (gtouch[i]) {
            if (gridDim.y == 1)
                gq[qa + i] += gacc[i];
            else
                atomicAdd(&gq[qa + i], gacc[i]);
        }
}

template <typename F>
hipError_t set_lds(F *kernel, size_t bytes)
{
    return allow_lds(reinterpret_cast<const void *>(kernel), bytes);
}

// Workgroups of `kernel` (kAccThreads threads, `lds` bytes of dynamic LDS) the device holds
// at once, looked up once per (device, kernel, lds).
template <typename F>
hipError_t resident_workgroups(F *kernel, size_t lds, int64_t *out)
{
    static std::mutex mu;
    static std::map<std::tuple<int, const void *, size_t>, int64_t> known;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    std::lock_guard<std::mutex> lock(mu);
    const auto key = std::make_tuple(dev, reinterpret_cast<const void *>(kernel), lds);
    auto it = known.find(key);
    if (it == known.end()) {
        int per_cu = 0, cus = 0;
        if ((e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, kAccThreads, lds)) != hipSuccess)
            return e;
        if ((e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess)
            return e;
        it = known.emplace(key, std::max<int64_t>(1, (int64_t)per_cu * cus)).first;
    }
    *out = it->second;
    return hipSuccess;
}

// Query slots per work item of a one-query launch: `want`, halved while the launch would hold
// fewer than kItemsMin items; at most 64 (an item's queries sit one per lane).
constexpr int64_t kItemsMin = 4096;
int32_t item_run(int32_t want, int64_t n_slots, int64_t n_tiles)
{
    int64_t run = want > 0 ? std::min<int64_t>(want, kWave) : 12;
    while (run > 1 && n_tiles * ((n_slots + run - 1) / run) < kItemsMin) run >>= 1;
    return (int32_t)run;
}

template <int VT, int B, bool SAMPLE>
hipError_t run_accumulate(const DevIndex &ix, const DevQueries &q, const DevCoarse &c,
                          const DevSlots &slots, int32_t n_sample, float *maxima,
                          const float *theta, const int32_t *sum_min, uint32_t *count, uint64_t *cand,
                          int64_t cap, int32_t per_item, int32_t max_terms, unsigned long long *queue,
                          hipStream_t s)
{
    const int eb = entry_block(B, max_terms);
    const size_t lds = accumulate_lds_bytes(B, ix.tile_stride, eb);
    hipError_t e;
    if constexpr (B == 1)
        e = set_lds(k_accumulate1<VT, SAMPLE>, lds);
    else
        e = set_lds(k_accumulate<VT, B, SAMPLE>, lds);
    if (e != hipSuccess) return e;
    const int64_t n_iter = SAMPLE ? n_sample : ix.n_tiles;
    if constexpr (B == 1) {
        AccArgs args{ix, q, c, slots, n_sample, maxima, theta, sum_min, count, cand, cap, {}, queue};
        AccItems &items = args.items;
        items.tiles = (uint32_t)n_iter;
        items.queues = 1;
        items.run = item_run(per_item, slots.n, n_iter);
        items.groups = (slots.n + items.run - 1) / items.run;
        items.n = n_iter * items.groups;
        if (queue) {  // one persistent launch over the items
            if ((e = set_lds(k_accumulate1_queue<VT, SAMPLE>, lds)) != hipSuccess) return e;
            int64_t wgs = 0;
            if ((e = resident_workgroups(k_accumulate1_queue<VT, SAMPLE>, lds, &wgs)) != hipSuccess)
                return e;
            // every queue then holds at least 4/15 of the workgroups' number in items, an eighth start on it
            if (n_iter >= kQueues && items.n >= 4 * wgs) items.queues = kQueues;
            hipLaunchKernelGGL((k_accumulate1_queue<VT, SAMPLE>), dim3((unsigned)std::min(wgs, items.n)),
                               dim3(kAccThreads), lds, s, args);
            return hipGetLastError();
        }
        // A grid dimension holds less than 2^32 threads, and one that exceeds that is cut off without
        // an error (8.4 million items of 512 threads), the second and third 65,535 workgroups.
        if ((int64_t)items.groups * kAccThreads > (int64_t)UINT32_MAX) return hipErrorInvalidValue;
        const int64_t rows = std::min<int64_t>(n_iter, 65535);
        hipLaunchKernelGGL((k_accumulate1<VT, SAMPLE>),
                           dim3((unsigned)items.groups, (unsigned)rows, (unsigned)((n_iter + rows - 1) / rows)),
                           dim3(kAccThreads), lds, s, args);
    } else {
        const int64_t n_batches = (slots.n + B - 1) / B;
        // Contiguous tile ranges per workgroup (see the kernel); the range length
        // keeps the grid at least a few times the chip's resident workgroups.
        int64_t per = per_item > 0 ? per_item : 12;
        while (per > 1 && n_batches * ((n_iter + per - 1) / per) < 4096) per >>= 1;
        int64_t groups = (n_iter + per - 1) / per;
        if (groups > 65535) {
            groups = 65535;
            per = (n_iter + groups - 1) / groups;
            groups = (n_iter + per - 1) / per;
        }
        hipLaunchKernelGGL((k_accumulate<VT, B, SAMPLE>), dim3((unsigned)n_batches, (unsigned)groups),
                           dim3(kAccThreads), lds, s, ix, q, c, slots, n_sample, maxima, theta, count,
                           cand, cap, (int32_t)per, (int32_t)eb);
    }
    return hipGetLastError();
}

template <int VT, bool SAMPLE>
hipError_t dispatch_b(int batch, const DevIndex &ix, const DevQueries &q, const DevCoarse &c,
                      const DevSlots &slots, int32_t n_sample, float *maxima,
                      const float *theta, const int32_t *sum_min, uint32_t *count, uint64_t *cand, int64_t cap,
                      int32_t per_item, int32_t max_terms, unsigned long long *queue,
                      hipStream_t s)
{
    switch (batch) {
    case 1: return run_accumulate<VT, 1, SAMPLE>(ix, q, c, slots, n_sample, maxima, theta, sum_min, count, cand, cap, per_item, max_terms, queue, s);
    case 2: return run_accumulate<VT, 2, SAMPLE>(ix, q, c, slots, n_sample, maxima, theta, sum_min, count, cand, cap, per_item, max_terms, nullptr, s);
    case 4: return run_accumulate<VT, 4, SAMPLE>(ix, q, c, slots, n_sample, maxima, theta, sum_min, count, cand, cap, per_item, max_terms, nullptr, s);
    case 8: return run_accumulate<VT, 8, SAMPLE>(ix, q, c, slots, n_sample, maxima, theta, sum_min, count, cand, cap, per_item, max_terms, nullptr, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t allow_lds(const void *kernel, size_t bytes)
{
    static std::mutex mu;
    static std::map<std::pair<int, const void *>, size_t> limit;  // (device, kernel) -> bytes
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    std::lock_guard<std::mutex> lock(mu);
    auto it = limit.find({dev, kernel});
    if (it == limit.end()) {
        int max = 0;
        hipFuncAttributes fa{};
        if ((e = hipDeviceGetAttribute(&max, hipDeviceAttributeMaxSharedMemoryPerBlock, dev)) != hipSuccess)
            return e;
        if ((e = hipFuncGetAttributes(&fa, kernel)) != hipSuccess) return e;
        const size_t lim = (size_t)max > fa.sharedSizeBytes ? (size_t)max - fa.sharedSizeBytes : 0;
        if ((e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lim)) !=
            hipSuccess)
            return e;
        it = limit.emplace(std::make_pair(dev, kernel), lim).first;
    }
    return bytes <= it->second ? hipSuccess : hipErrorInvalidValue;
}

hipError_t launch_query_prep(const DevQueries &q, int64_t n_cols, double beta, DevCoarse c,
                             const float *term_max, double *scratch_abs, int32_t *err_flag,
                             uint32_t *zero, int64_t n_zero, hipStream_t s)
{
    if (q.n_rows == 0) return hipSuccess;
    dim3 grid((unsigned)((q.n_rows + kPrepWaves - 1) / kPrepWaves));
    if (grid.x > 1) {
        const hipError_t e = launch_fill_u32(reinterpret_cast<uint32_t *>(err_flag), 4, 0u, s);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_query_prep, grid, dim3(kPrepWaves * kWave), 0, s, q, n_cols, beta, c, term_max,
                       scratch_abs, err_flag, zero, n_zero);
    return hipGetLastError();
}

hipError_t launch_accumulate(const DevIndex &ix, const DevQueries &q, const DevCoarse &c,
                             int batch, bool sample, const DevSlots &slots,
                             int32_t n_sample_tiles, float *maxima, const float *theta,
                             const int32_t *sum_min, uint32_t *count, uint64_t *cand, int64_t cap,
                             int32_t per_item, int32_t max_terms, unsigned long long *queue,
                             hipStream_t s)
{
    if (slots.n == 0 || ix.n_tiles == 0) return hipSuccess;
    const int vt = ix.value_dtype;
    if (sample) {
        if (vt == 0) return dispatch_b<0, true>(batch, ix, q, c, slots, n_sample_tiles, maxima, theta, sum_min, count, cand, cap, per_item, max_terms, queue, s);
        if (vt == 1) return dispatch_b<1, true>(batch, ix, q, c, slots, n_sample_tiles, maxima, theta, sum_min, count, cand, cap, per_item, max_terms, queue, s);
        return dispatch_b<2, true>(batch, ix, q, c, slots, n_sample_tiles, maxima, theta, sum_min, count, cand, cap, per_item, max_terms, queue, s);
    }
    if (vt == 0) return dispatch_b<0, false>(batch, ix, q, c, slots, n_sample_tiles, maxima, theta, sum_min, count, cand, cap, per_item, max_terms, queue, s);
    if (vt == 1) return dispatch_b<1, false>(batch, ix, q, c, slots, n_sample_tiles, maxima, theta, sum_min, count, cand, cap, per_item, max_terms, queue, s);
    return dispatch_b<2, false>(batch, ix, q, c, slots, n_sample_tiles, maxima, theta, sum_min, count, cand, cap, per_item, max_terms, queue, s);
}

// Selecting kernels (k_theta, k_finalize): large workgroups while they all run at once, small ones
// beyond (kFewSlots = two 1,024-thread workgroups per CU).  Threshold of one query: 4.7 us with
// 1,024 threads, 8.7 with 256; of 1,000 queries: 12.4 and 11.2 us.
constexpr int32_t kFewSlots = 512;

hipError_t launch_theta(const float *maxima, int64_t n_maxima, int64_t rank, const DevSlots &slots,
                        const float *qinv, float *theta, int32_t *sum_min, hipStream_t s)
{
    if (slots.n == 0) return hipSuccess;
    if (slots.n <= kFewSlots)
        hipLaunchKernelGGL((k_theta<1024, 4>), dim3((unsigned)slots.n), dim3(1024), 0, s, maxima,
                           n_maxima, rank, slots, qinv, theta, sum_min);
    else
        hipLaunchKernelGGL((k_theta<256, 16>), dim3((unsigned)slots.n), dim3(256), 0, s, maxima,
                           n_maxima, rank, slots, qinv, theta, sum_min);
    return hipGetLastError();
}

hipError_t launch_fill_f32(float *p, int64_t n, float v, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    int64_t blocks = (n + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(k_fill_f32, dim3((unsigned)blocks), dim3(256), 0, s, p, n, v);
    return hipGetLastError();
}
hipError_t launch_fill_u32(uint32_t *p, int64_t n, uint32_t v, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    int64_t blocks = (n + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)blocks), dim3(256), 0, s, p, n, v);
    return hipGetLastError();
}

hipError_t launch_report(const DevRetry &r, hipStream_t s)
{
    hipLaunchKernelGGL(k_report, dim3(1), dim3(1), 0, s, r);
    return hipGetLastError();
}

hipError_t launch_finalize(const DevIndex &ix, const DevQueries &q, const DevSlots &slots,
                           const uint32_t *count, const uint64_t *cand,
                           const float *theta, int64_t cap, int32_t need, int32_t k, bool rerank,
                           int32_t max_qnnz, uint64_t *pool, int64_t *out_ids, float *out_scores,
                           const DevRetry &retry, hipStream_t s)
{
    const int32_t n_slots = slots.n;
    if (n_slots == 0) return hipSuccess;
    // bitmap of candidate ids below need + cap: zero-score documents in id order
    const int64_t bm = theta ? (need + cap + 31) / 32 : 0;
    if (bm > (int64_t)1 << 20) return hipErrorInvalidValue;
    // Keys and bitmap may take the LDS but for 1,056 bytes, 1,024 of them beside the kernel's own: a
    // pool of 500 takes candidate buffers of up to 1,269,004 entries.  (With the select's tables in
    // LDS of their own it was 9,344 fewer.)
    constexpr size_t kSpare = 1024;
    const size_t keys = (size_t)pow2_at_least(need) * 8;
    const size_t lds = keys + std::max((size_t)bm * 4, sizeof(SelectLds));
    if (rerank && !pool) return hipErrorInvalidValue;
    hipError_t e;
    auto finalize = [&](auto kernel, int nt) -> hipError_t {
        hipError_t r = set_lds(kernel, std::max(lds, keys + (size_t)bm * 4 + kSpare));
        if (r != hipSuccess) return r;
        hipLaunchKernelGGL(kernel, dim3((unsigned)n_slots), dim3(nt), lds, s, ix, slots, count,
                           cand, theta, cap, need, k, (int32_t)bm, pool, out_ids, out_scores, retry);
        return hipGetLastError();
    };
    // 1,024 threads where every document is a candidate (10,000 of them: 8.3 us, 20 us with 256
    // threads); a threshold leaves one or two thousand, which 256 threads select sooner (one query
    // 5.9 against 6.4 us, 37 queries 7.8 against 9.6)
    const bool wide = n_slots <= kFewSlots && !theta;
    if (!rerank) {
        e = wide ? finalize(k_finalize<false, 1024, 8>, 1024) : finalize(k_finalize<false, 256, 8>, 256);
        return e != hipSuccess ? e : launch_report(retry, s);
    }
    e = wide ? finalize(k_finalize<true, 1024, 8>, 1024) : finalize(k_finalize<true, 256, 8>, 256);
    if (e != hipSuccess) return e;
    const int32_t tlg = table_lg(max_qnnz > 0 ? max_qnnz : 1);
    const size_t lds_t = (size_t)16 << tlg;
    e = set_lds(k_rerank, lds_t);
    if (e != hipSuccess) return e;
    // few queries: fewer entries per workgroup, so that more of them share the work
    constexpr int kPerGroup = kFinThreads / kWave * kRerankPerWave;
    int32_t groups = kRerankGroups;
    while (groups > 1 && (int64_t)n_slots * ((need + kPerGroup * groups - 1) / (kPerGroup * groups)) < kRerankFill)
        groups >>= 1;
    const unsigned blocks = (unsigned)((need + kPerGroup * groups - 1) / (kPerGroup * groups));
    hipLaunchKernelGGL(k_rerank, dim3((unsigned)n_slots, blocks), dim3(kFinThreads), lds_t, s, ix,
                       q, slots, need, tlg, groups, pool, retry);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    auto topk = [&](auto kernel, size_t bytes) -> hipError_t {
        hipError_t r = set_lds(kernel, bytes);
        if (r != hipSuccess) return r;
        hipLaunchKernelGGL(kernel, dim3((unsigned)n_slots), dim3(kFinThreads), bytes, s, slots,
                           need, k, pool, out_ids, out_scores, retry);
        return hipGetLastError();
    };
    if (k < need && k <= kRankSort && need > kRankSort && need <= kFinThreads * kTopkRegs)
        return topk(k_topk<true>, (size_t)pow2_at_least(k) * 8);
    return topk(k_topk<false>, keys);
}

namespace {
// Row groups per wave of a pair-score launch: fewer where the workgroups would not fill the
// chip, more where the grid's second dimension would not hold them.
int32_t score_groups(int64_t n_rows, int64_t n_cand)
{
    constexpr int64_t kPer = kFinThreads / kWave * 4;
    int64_t g = kRerankGroups;
    while (g > 1 && n_rows * ((n_cand + kPer * g - 1) / (kPer * g)) < kRerankFill) g >>= 1;
    while ((n_cand + kPer * g - 1) / (kPer * g) > 65535) g <<= 1;
    return (int32_t)g;
}
dim3 score_grid(int64_t n_rows, int64_t n_cand, int32_t groups)
{
    const int64_t per = (int64_t)(kFinThreads / kWave) * 4 * groups;
    return dim3((unsigned)n_rows, (unsigned)((n_cand + per - 1) / per));
}
}  // namespace

hipError_t launch_score_forward(const DevIndex &ix, const DevQueries &q, const int64_t *cand,
                                int32_t n_cand, int32_t max_qnnz, float *out, hipStream_t s)
{
    if (q.n_rows == 0 || n_cand == 0) return hipSuccess;
    const int32_t tlg = table_lg(max_qnnz), groups = score_groups(q.n_rows, n_cand);
    const size_t lds = (size_t)16 << tlg;
    hipError_t e = set_lds(k_score_forward, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_score_forward, score_grid(q.n_rows, n_cand, groups), dim3(kFinThreads),
                       lds, s, ix, q, cand, n_cand, tlg, groups, out);
    return hipGetLastError();
}

hipError_t launch_score_backward(const DevIndex &ix, const DevQueries &q, const int64_t *cand,
                                 int32_t n_cand, int32_t max_qnnz, const float *grad, float *gq,
                                 float *gx, hipStream_t s)
{
    if (q.n_rows == 0 || n_cand == 0 || (!gq && !gx)) return hipSuccess;
    const int32_t tlg = table_lg(max_qnnz), groups = score_groups(q.n_rows, n_cand);
    const size_t lds = ((size_t)16 << tlg) + (size_t)max_qnnz * 12;
    hipError_t e = set_lds(k_score_backward, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_score_backward, score_grid(q.n_rows, n_cand, groups), dim3(kFinThreads),
                       lds, s, ix, q, cand, n_cand, tlg, groups, grad, gq, gx);
    return hipGetLastError();
}

}  // namespace sindi
