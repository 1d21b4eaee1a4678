// Triangle counting: static count and the delta for a batch (undirected graphs).
//
// Delta (Appendix A, DynTC: Decremental runs on the old graph, Incremental on the
// new one).  For a changed edge {a, b} every common neighbour c closes a
// triangle {a, b, c}; if k of that triangle's three edges are in the batch, the
// triangle is met once from each of them, so each meeting adds 6 / k and the sum
// over all changed edges is 6x the number of changed triangles -- the listing's
// count1/2 + count2/4 + count3/6 with every edge taken once instead of twice.
// An edge is "in the batch" when its entry carries MARK: deletions carry it
// between marking and commit (so the old graph still holds them), insertions
// from insertion until the post-hooks are done -- the edge flags modified_del /
// modified_add of the listing.
//
// Static (comparator; Appendix A staticTC counts every triangle once by vertex
// order): here vertices are ranked by (degree, id), every edge is oriented from
// its lower- to its higher-ranked end, and a triangle is counted once at its
// lowest-ranked vertex by intersecting two forward lists -- the standard forward
// algorithm, whose degree ordering bounds every forward list by sqrt(2m) on skewed
// graphs.
#include <algorithm>
#include <type_traits>

#include "dg_device.h"

namespace dg {

static inline int grid_for(int64_t n) {
    int64_t g = (n + 255) / 256;
    return (int)(g < 1 ? 1 : (g > 8192 ? 8192 : g));
}

// Blocks of WIDE_T threads (kernels that add into one shared counter).
static inline int grid_wide(int64_t n) {
    const int64_t g = (n + WIDE_T - 1) / WIDE_T;
    return (int)(g < 1 ? 1 : (g > 512 ? 512 : g));
}

// A value that is the same in every lane, in scalar registers.
__device__ __forceinline__ int64_t wave_first(int64_t v) {
    return (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(v >> 32)) << 32) |
                     (uint32_t)__builtin_amdgcn_readfirstlane((int)v));
}

struct RowRef {
    int64_t ob, db, od, dd;  // base start/len, diff start/len
};

__device__ __forceinline__ RowRef row_ref(const int64_t *off, const int64_t *doff, int32_t v) {
    RowRef r;
    r.ob = off[v];
    r.db = off[v + 1] - r.ob;
    r.od = doff[v];
    r.dd = doff[v + 1] - r.od;
    return r;
}

// Live entry for neighbour x in row r: returns the raw entry (flags) or 0 with
// found = false.
__device__ __forceinline__ bool row_find(const int32_t *col, const int32_t *dcol, const RowRef &r,
                                         uint32_t x, uint32_t &ent) {
    int64_t p = find_sorted(col, r.ob, r.ob + r.db, x);
    if (p >= 0) {
        ent = (uint32_t)col[p];
        return !(ent & DEAD);
    }
    if (r.dd > 0) {
        int64_t q = find_sorted(dcol, r.od, r.od + r.dd, x);
        if (q >= 0) {
            ent = (uint32_t)dcol[q];
            return !(ent & DEAD);
        }
    }
    return false;
}

// Fenced search of a long base row: every stride-th neighbour id of the row is
// copied to LDS once per work item (stride: the smallest power of two from
// TC_FSTRIDE_MIN that needs at most TC_FCAP fences); a probe searches those
// fences in LDS and then only the stride-entry segment they select in global
// memory.  Rows of at most TC_FMIN entries, or longer than TC_FCAP *
// TC_FSTRIDE_MAX, are searched whole.
constexpr int TC_FSTRIDE_MIN = 8;
constexpr int TC_FSTRIDE_MAX = 2048;
constexpr int TC_FCAP = 128;  // fences per wave (rows up to 262,144 entries are fenced)
constexpr int TC_FMIN = 128;

// Searches of the neighbours x[u] in a sorted row of len entries: e[u] becomes the entry
// (with its flags) of x[u] if the row has one, else some other entry.  Each starts
// at s[u], with e[u] there, and covers the next size entries (a power of two); the steps go
// side by side, so that U gathers are in flight per lane instead of one, and the last four
// entries are read at once.
struct __attribute__((packed, aligned(4))) Four {
    uint32_t e[4];
};
template <int U>
__device__ __forceinline__ void find_step(const int32_t *__restrict__ row, uint32_t len, int size,
                                          const uint32_t (&x)[U], uint32_t (&s)[U], uint32_t (&e)[U]) {
    const bool four = size >= 4 && len >= 4;
    for (int h = size >> 1; h > (four ? 2 : 0); h >>= 1) {
        uint32_t y[U];
#pragma unroll
        for (int u = 0; u < U; ++u) y[u] = (uint32_t)row[min(s[u] + h, len - 1)];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool go = s[u] + h < len && (y[u] & ID_MASK) <= x[u];
            s[u] += go ? h : 0;
            e[u] = go ? y[u] : e[u];
        }
    }
    if (!four) return;
    Four y[U];
#pragma unroll
    for (int u = 0; u < U; ++u) y[u] = *reinterpret_cast<const Four *>(row + min(s[u], len - 4));
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if ((y[u].e[k] & ID_MASK) == x[u]) e[u] = y[u].e[k];
}

// The start of find_step from a row's fences, f[k] = entry k * stride for k < nf.  False
// if every x of the wave lies below the row.
template <int U>
__device__ __forceinline__ bool find_fenced(const uint32_t *f, int nf, int stride, const uint32_t (&xs)[U],
                                            uint32_t (&s)[U], uint32_t (&e)[U]) {
    // one search would begin with: if (x < f[0]) return -1;  a wave leaves if every lane would
    const uint32_t head = f[0] & ID_MASK;
    bool some = false;
#pragma unroll
    for (int u = 0; u < U; ++u) some |= xs[u] >= head;
    if (ballot(some) == 0) return false;
    int top = 1;
    while (top < nf) top <<= 1;
#pragma unroll
    for (int u = 0; u < U; ++u) s[u] = 0;
    for (int h = top >> 1; h > 0; h >>= 1) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t k = min(s[u] + h, (uint32_t)(nf - 1));
            if ((f[k] & ID_MASK) <= xs[u]) s[u] = k;
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        e[u] = f[s[u]];
        s[u] *= stride;
    }
    return true;
}

// Per-block partials (no contended atomics; summed in block order by k_tc_sum): 6 x the
// changed triangles, the entries walked, and the other words of 4 bytes read (row bounds
// and search steps).
__device__ __forceinline__ void tc_block_part(uint64_t acc, uint64_t walked, uint64_t probes, int64_t *part) {
    __shared__ uint64_t s_p[3][256 / WAVE];
    acc = wave_sum(acc);
    walked = wave_sum(walked);
    probes = wave_sum(probes);
    const int wv = threadIdx.x / WAVE;
    if (lane_id() == 0) {
        s_p[0][wv] = acc;
        s_p[1][wv] = walked;
        s_p[2][wv] = probes;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        uint64_t s = 0;
        for (int q = 0; q < (int)blockDim.x / WAVE; ++q) s += s_p[threadIdx.x][q];
        part[3 * (int64_t)blockIdx.x + threadIdx.x] = (int64_t)s;
    }
}

// Reads of a binary search of len entries.
__device__ __forceinline__ int search_steps(int64_t len) {
    return len > 0 ? 64 - __clzll((unsigned long long)len) : 0;
}

// Work items: a changed edge's shorter row is cut into pieces of TC_CHUNK entries,
// so that an edge between two hubs (tens of thousands of common candidates) is
// spread over many waves instead of holding one wave for the whole launch.
constexpr int TC_CHUNK = 256;
constexpr uint32_t ABSENT = ~0u;  // no entry: dead, and of no id

// cnt[i] = pieces of changed edge i (0 when its shorter row is empty); cnt[ne] = 0.
// Edges of at most TC_SHORT candidates are finished here and get no pieces: a wave takes
// TC_WINDOW edges and its lanes take their candidates in turn, each searching its own edge's
// longer row.  As work items of their own, a few candidates each, they left most lanes
// idle over the whole chain of dependent reads (1M vertices, 84k new edges with 230k
// candidates: 6 + 80 us for this launch and the next, now 23 + 16).
constexpr int TC_SHORT = 32, TC_WINDOW = 16;

__global__ __launch_bounds__(256) void k_tc_items(int64_t ne, const int32_t *__restrict__ eu,
                                                  const int32_t *__restrict__ ev, const int64_t *__restrict__ off,
                                                  const int32_t *__restrict__ col, const int64_t *__restrict__ doff,
                                                  const int32_t *__restrict__ dcol, int64_t *cnt, int64_t *part) {
    const int l = lane_id();
    uint64_t acc = 0, walked = 0, probes = 0;
    const int64_t nwaves = gstride() / WAVE;
    for (int64_t w = gtid() / WAVE; w * TC_WINDOW <= ne; w += nwaves) {
        const int64_t i = w * TC_WINDOW + l;
        int64_t ta = 0, tb = 0;
        int32_t a = 0, b = 0;  // the rows' vertices, the shorter first
        if (l < TC_WINDOW && i < ne) {
            a = eu[i];
            b = ev[i];
            ta = (off[a + 1] - off[a]) + (doff[a + 1] - doff[a]);
            tb = (off[b + 1] - off[b]) + (doff[b + 1] - doff[b]);
            if (ta > tb) {
                int32_t v = a;
                a = b;
                b = v;
                ta = tb;
            }
        }
        const int mine = ta <= TC_SHORT ? (int)ta : 0;
        if (l < TC_WINDOW && i <= ne) cnt[i] = mine ? 0 : (ta + TC_CHUNK - 1) / TC_CHUNK;
        int upto = mine;  // candidates of the lanes up to this one
#pragma unroll
        for (int d = 1; d < TC_WINDOW; d <<= 1) {
            const int y = __shfl_up(upto, d, WAVE);
            if (l >= d) upto += y;
        }
        const int total = __shfl(upto, TC_WINDOW - 1, WAVE);
        for (int e0 = 0; e0 < total; e0 += WAVE) {
            const int e = min(e0 + l, total - 1);
            int k = 0;  // the first edge whose candidates reach past e
#pragma unroll
            for (int h = TC_WINDOW / 2; h > 0; h >>= 1)
                if (__shfl(upto, k + h - 1, WAVE) <= e) k += h;
            const int j = e - (__shfl(upto, k, WAVE) - __shfl(mine, k, WAVE));
            const int32_t sv = __shfl(a, k, WAVE), lv = __shfl(b, k, WAVE);
            const RowRef ra = row_ref(off, doff, sv), rb = row_ref(off, doff, lv);
            const uint32_t x = j < ra.db ? (uint32_t)col[ra.ob + j] : (uint32_t)dcol[ra.od + (j - ra.db)];
            if (e0 + l >= total) continue;
            probes += search_steps(rb.db) + search_steps(rb.dd);
            if (x & DEAD) continue;
            uint32_t x2;
            if (!row_find(col, dcol, rb, x & ID_MASK, x2)) continue;
            acc += (uint64_t)(6 / (1 + ((x & MARK) ? 1 : 0) + ((x2 & MARK) ? 1 : 0)));
        }
        if (l < TC_WINDOW && i < ne) probes += 8;
        if (l == 0) walked += total;
    }
    tc_block_part(acc, walked, probes, part);
}

// One wave per work item; lanes walk the item's piece of the smaller row and probe
// the larger one.  start = exclusive scan of the piece counts (start[ne] = total).
// The gathers of the searches bound it, one line per lane and step (R-MAT 20 without 84k
// of its edges, 39M candidates: 77 % of the time).  With one candidate per lane it waited for
// each step instead, 500 us a launch; with a piece's four side by side 350, and with the
// last two steps read as one group of four entries 325.  (More fences cost as much to
// read as they save; pieces of 128 took 445 us.)
__global__ __launch_bounds__(256) void k_tc_delta(int64_t ne, const int32_t *eu, const int32_t *ev,
                                                  const int64_t *__restrict__ start,
                                                  const int64_t *__restrict__ off,
                                                  const int32_t *__restrict__ col,
                                                  const int64_t *__restrict__ doff,
                                                  const int32_t *__restrict__ dcol, int64_t *part) {
    __shared__ uint32_t s_fence[256 / WAVE][TC_FCAP];
    const int64_t wave_global = wave_first(((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / WAVE);
    const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) / WAVE;
    const int l = lane_id();
    uint32_t *f = s_fence[threadIdx.x / WAVE];
    uint64_t acc = 0, walked = 0, probes = 0;
    const int64_t items = start[ne];
    for (int64_t it = wave_global; it < items; it += nwaves) {
        // the edge of item it: start[i] <= it < start[i + 1], found by a 64-way
        // search (each lane probes one point, a ballot keeps the prefix at or below it)
        int64_t lo = 0, hi = ne;  // start[lo] <= it < start[hi]
        while (hi - lo > 1) {
            const int64_t step = (hi - lo + WAVE - 1) / WAVE;
            const int64_t p = lo + (int64_t)(l + 1) * step;
            const uint64_t le = __ballot(p < hi && start[p] <= it);
            lo += (int64_t)__popcll(le) * step;
            hi = min(hi, lo + step);
        }
        const int64_t i = wave_first(lo), piece = it - start[i];  // (the same in every lane: scalar from here)
        int32_t a = eu[i], b = ev[i];
        RowRef ra = row_ref(off, doff, a), rb = row_ref(off, doff, b);
        if (ra.db + ra.dd > rb.db + rb.dd) {
            RowRef t = ra; ra = rb; rb = t;
        }
        const int64_t j0 = piece * TC_CHUNK, j1 = min(ra.db + ra.dd, j0 + TC_CHUNK);
        int stride = TC_FSTRIDE_MIN;
        while ((int64_t)stride * TC_FCAP < rb.db && stride < TC_FSTRIDE_MAX) stride <<= 1;
        const int64_t nf64 = (rb.db + stride - 1) / stride;
        const bool fenced = j1 > j0 && rb.db > TC_FMIN && nf64 <= TC_FCAP;
        const int nf = fenced ? (int)nf64 : 0;
        if (fenced) {
            wave_sync();  // every lane is done with the previous edge's fences
            for (int k = l; k < nf; k += WAVE) f[k] = (uint32_t)col[rb.ob + (int64_t)k * stride];
            wave_sync();
        }
        // global reads of one probe: the whole binary search, or the segment's
        const int depth = search_steps(fenced ? stride : rb.db) + search_steps(rb.dd);
        if (l == 0) {
            walked += (j1 - j0) + nf;
            probes += (j1 - j0) * depth + (piece == 0 ? 8 : 0);
        }
        const int32_t *row = col + rb.ob, *drow = dcol + rb.od;
        int whole = 1, dwhole = 1;  // powers of two that cover the rows
        while (whole < rb.db) whole <<= 1;
        while (dwhole < rb.dd) dwhole <<= 1;
        // U candidates per lane, 64 apart
        const auto probe = [&](auto uc, int64_t j) {
            constexpr int U = decltype(uc)::value;
            uint32_t e[U], c[U], s[U], e2[U];
#pragma unroll
            for (int u = 0; u < U; ++u, j += WAVE) {
                const int64_t k = min(j, j1 - 1);
                e[u] = (uint32_t)*(k < ra.db ? col + ra.ob + k : dcol + ra.od + (k - ra.db));
                if (j >= j1) e[u] = DEAD;
                c[u] = e[u] & ID_MASK;
                e2[u] = ABSENT;
                s[u] = 0;
            }
            if (rb.db > 0) {
                if (fenced) {
                    if (find_fenced<U>(f, nf, stride, c, s, e2)) find_step<U>(row, rb.db, stride, c, s, e2);
                } else {
#pragma unroll
                    for (int u = 0; u < U; ++u) e2[u] = (uint32_t)row[0];
                    find_step<U>(row, rb.db, whole, c, s, e2);
                }
            }
            if (rb.dd > 0) {
                uint32_t d2[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    s[u] = 0;
                    d2[u] = (uint32_t)drow[0];
                }
                find_step<U>(drow, rb.dd, dwhole, c, s, d2);
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if ((e2[u] & ID_MASK) != c[u]) e2[u] = d2[u];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const bool hit = (e2[u] & ID_MASK) == c[u] && !((e[u] | e2[u]) & DEAD);
                const int k = 1 + ((e[u] & MARK) ? 1 : 0) + ((e2[u] & MARK) ? 1 : 0);
                acc += hit ? (uint64_t)(6 / k) : 0;
            }
        };
        if (j1 <= j0) continue;
        if (j1 - j0 <= WAVE) probe(std::integral_constant<int, 1>(), j0 + l);
        else probe(std::integral_constant<int, TC_CHUNK / WAVE>(), j0 + l);
    }
    tc_block_part(acc, walked, probes, part);
}

// Sums of the per-block partials: block 0 those of nblocks blocks of k_tc_delta, block 1
// those of the niblocks blocks of k_tc_items that follow them.
__global__ __launch_bounds__(1024) void k_tc_sum(const int64_t *part, int64_t nblocks, int64_t niblocks, int64_t *out,
                                                 int64_t *iout) {
    __shared__ int64_t s[3][1024 / WAVE];
    int64_t a0 = 0, a1 = 0, a2 = 0;
    if (blockIdx.x == 1) {
        part += 3 * nblocks;
        nblocks = niblocks;
        out = iout;
    }
    for (int64_t b = threadIdx.x; b < nblocks; b += blockDim.x) {
        a0 += part[3 * b];
        a1 += part[3 * b + 1];
        a2 += part[3 * b + 2];
    }
    a0 = wave_sum(a0);
    a1 = wave_sum(a1);
    a2 = wave_sum(a2);
    const int wv = threadIdx.x / WAVE;
    if (lane_id() == 0) {
        s[0][wv] = a0;
        s[1][wv] = a1;
        s[2][wv] = a2;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        int64_t a = 0;
        for (int q = 0; q < (int)blockDim.x / WAVE; ++q) a += s[threadIdx.x][q];
        out[threadIdx.x] = a;
    }
}

int tc_delta(dg_graph *g, const int32_t *eu, const int32_t *ev, int64_t ne, uint64_t *sum6, int64_t *entries) {
    *sum6 = 0;
    if (entries) *entries = 0;
    if (ne <= 0) return DG_OK;
    hipStream_t s = g->stream;
    Dir &F = g->fwd;
    // four waves per block; 16,384, 8,192 and 4,096 blocks: 310, 320 and 340 us where the
    // items are many, 30, 16 and 12 us where they are few
    int64_t blocks = std::min<int64_t>((ne + 3) / 4, 8192);
    const int64_t iblocks = std::min<int64_t>((ne / TC_WINDOW + 4) / 4, 8192);
    DG_TRY(g->ws.bpart.ensure(3 * (size_t)(blocks + iblocks) + 8));
    DG_TRY(g->ws.tcitems.ensure(2 * ((size_t)ne + 1)));
    int64_t *cnt = g->ws.tcitems.p, *start = g->ws.tcitems.p + ne + 1;
    const int pi = prof_begin("tc_items", s);
    hipLaunchKernelGGL(k_tc_items, dim3((unsigned)iblocks), dim3(256), 0, s, ne, eu, ev, F.off.p, F.col.p, F.doff.p,
                       F.dcol.p, cnt, g->ws.bpart.p + 3 * blocks);
    prof_end(pi, s, 0.0);
    DG_HIP(hipGetLastError());
    DG_TRY(scan_excl(g, cnt, start, ne + 1));
    const int ps = prof_begin("tc_delta", s);
    hipLaunchKernelGGL(k_tc_delta, dim3((unsigned)blocks), dim3(256), 0, s, ne, eu, ev, start, F.off.p, F.col.p,
                       F.doff.p, F.dcol.p, g->ws.bpart.p);
    prof_end(ps, s, 0.0);
    static_assert(C_AUX2 == C_AUX1 + 1 && C_AUX3 == C_AUX1 + 2 && C_RED0 + 3 <= C_EDGES, "three consecutive counters");
    hipLaunchKernelGGL(k_tc_sum, dim3(2), dim3(1024), 0, s, g->ws.bpart.p, blocks, iblocks, g->ws.dcnt + C_AUX1,
                       g->ws.dcnt + C_RED0);
    DG_HIP(hipGetLastError());
    DG_TRY(counters_read(g));
    const int64_t *delta = g->ws.hcnt + C_AUX1, *items = g->ws.hcnt + C_RED0;
    *sum6 = (uint64_t)(delta[0] + items[0]);
    if (entries) *entries = delta[1] + items[1];  // shorter-row entries intersected
    // of each launch: per changed edge that it looks at its endpoints' offsets (32 B); per
    // entry of the shorter row and per fence of a long row 4 B; per global search step into
    // the longer row (the whole row, or the segment a fence search selects) 4 B
    prof_add(pi, 4.0 * (double)(items[1] + items[2]));
    prof_add(ps, 4.0 * (double)(delta[1] + delta[2]));
    return DG_OK;
}

// ---- static count on a merged (plain CSR) graph -------------------------------------

__device__ __forceinline__ bool rank_lt(int32_t du, int32_t u, int32_t dv, int32_t v) {
    return du < dv || (du == dv && u < v);
}

// Forward (oriented) lists: N+(x) = the neighbours of x ranked above x, kept in id
// order.  One wave per row; pass 1 writes |N+(x)| to odeg, pass 2 fills ocol
// from the scanned offsets ooff (ballot compaction keeps the order).
template <bool FILL>
__global__ __launch_bounds__(256) void k_tc_orient(int32_t n, const int64_t *__restrict__ off,
                                                   const int32_t *__restrict__ col,
                                                   const int32_t *__restrict__ deg, int64_t *odeg,
                                                   const int64_t *__restrict__ ooff, int32_t *ocol) {
    const int64_t wave_global = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / WAVE;
    const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) / WAVE;
    const int l = lane_id();
    for (int64_t x = wave_global; x < n; x += nwaves) {
        const int64_t xs = off[x], xe = off[x + 1];
        const int32_t dx = deg[x];
        int64_t cnt = 0;
        const int64_t base = FILL ? ooff[x] : 0;
        for (int64_t j0 = xs; j0 < xe; j0 += WAVE) {
            const int64_t j = j0 + l;
            bool up = false;
            int32_t y = 0;
            if (j < xe) {
                const uint32_t c = (uint32_t)col[j];
                y = (int32_t)(c & ID_MASK);
                up = !(c & DEAD) && rank_lt(dx, (int32_t)x, deg[y], y);
            }
            const uint64_t b = ballot(up);
            if (FILL && up) ocol[base + cnt + __popcll(b & lanemask_lt())] = y;
            cnt += __popcll(b);
        }
        if (!FILL && l == 0) odeg[x] = cnt;
    }
}

// On a graph whose ids run in the order of falling degree (built so, and not changed
// since) the neighbours ranked above x, ties to the smaller id, are the entries of its row
// below x: the forward lists are the rows' beginnings where they stand, and only their
// ends pend[x] are needed.  *out_of_order becomes non-zero if a degree rises with the id;
// the lists are then built, because order by outdated degrees could leave a list
// as long as its row.  262k vertices, 8.4M entries: 12 us in place of 450 for the two
// passes of k_tc_orient and their scan.  *low counts the entries below x that are below
// `ids` too (k_tc_forward's choice).
__global__ __launch_bounds__(WIDE_T) void k_tc_prefix(int32_t n, const int64_t *__restrict__ off,
                                                      const int32_t *__restrict__ col,
                                                      const int32_t *__restrict__ deg, int32_t ids, int64_t *pend,
                                                      int64_t *out_of_order, int64_t *low) {
    __shared__ BlockScratch sc;
    const auto below = [&](int64_t lo, int64_t hi, uint32_t v) {
        while (lo < hi) {
            const int64_t mid = (lo + hi) >> 1;
            if (((uint32_t)col[mid] & ID_MASK) < v) lo = mid + 1;
            else hi = mid;
        }
        return lo;
    };
    bool bad = false;
    int64_t few = 0;
    for (int64_t x = gtid(); x < n; x += gstride()) {
        bad |= x + 1 < n && deg[x] < deg[x + 1];
        const int64_t s = off[x], e = below(s, off[x + 1], (uint32_t)x);
        pend[x] = e;
        few += (x <= ids ? e : below(s, e, (uint32_t)ids)) - s;
    }
    if (ballot(bad) != 0 && lane_id() == 0) *out_of_order = 1;
    block_count<WIDE_T>(low, few, sc);
}

// Every triangle, ranked a < b < c, is counted once: at x = a and y = b, as the
// common element c of N+(a) and N+(b).  One wave per row x copies N+(x) to LDS
// (when it fits) and walks y over N+(x).  For each y the lanes either stream
// N+(y) and look its elements up in the LDS copy (one coalesced load per 64 elements),
// or, when N+(y) is much longer, take the elements of N+(x) and binary-search N+(y)
// in memory (262k vertices, 4.2M edges: 620M lookups and 0.5M searched lists).
//
// BITS: forward lists of skewed graphs in the degree order point to vertices of higher
// degree, so most of their ids are small, and the copy is a bitmap of the ids below
// TCF_IDS: a lookup is one LDS read where the search of a sorted copy takes up to ten.
// Larger ids are searched in the list's tail in memory, which costs more than the sorted
// copy where many entries are large, so the bitmap is taken from TCF_LOW of the entries
// below TCF_IDS on (us a count with the bitmap and with the copy, lists in place:
// R-MAT 18 with 16 edges a vertex, share 0.99, 425 and 1516; R-MAT 22, 0.79, 6081 and 14310;
// a power law of 1M vertices, 0.65, 1283 and 1338; even degrees, 100k vertices, 0.61, 600
// and 543; 262k, 0.28, 2279 and 1334; 1M, 0.08, 10830 and 5135).  (A hash set of the same
// size was slower than either: 2.44 ms against 1.56 ms for the search; the bitmap took
// 0.80 ms, bound by the instructions around a lookup, and 0.41 ms with the lists whose ids
// are all in its range read by bits_hits.)
constexpr double TCF_LOW = 0.625;
constexpr int TCF_CAP = 1024;  // forward-list entries of a row staged in LDS, per wave
constexpr int TCF_IDS = 32 * TCF_CAP;
// Four or more grids of resident blocks, few enough adds to the total.  The copy's counts are
// longer and gain from shorter blocks: R-MAT 20 in the order given 90.9 and 74.2 ms with
// 8,192 and 32,768, the bitmap's R-MAT 18 425 and 604 us.
constexpr int TCF_BLOCKS = 8192, TCF_BLOCKS_COPY = 32768;

__device__ __forceinline__ bool lds_has(const int32_t *a, int len, int32_t v) {
    int lo = 0, hi = len;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (a[mid] < v) lo = mid + 1;
        else hi = mid;
    }
    return lo < len && a[lo] == v;
}

constexpr int TCF_LISTS = 4, TCF_LOADS = 2;  // lists together, and loads of each in flight
// A list more than this many times longer than N+(x) is searched: a search is ten dependent
// reads, a 64-entry step of the list about six instructions (6: 429 us, 16 to 64: 415)
constexpr int TCF_LONG = 16;

// How many entries of the lists of the lanes in `lists` (ys, len: bounds of a lane's list,
// all ids below TCF_IDS) are in the bitmap sx; summed over the lanes' results.
// The lists of a group are read through buffer descriptors of their lengths, which
// answer 0 past the end: neither addresses nor bounds cost vector instructions, and the
// zeros, looked up like any entry, are taken off at the end if id 0 is in the bitmap.
__device__ __forceinline__ uint64_t bits_hits(const int32_t *sx, const int32_t *ocol, int64_t ys, int32_t len,
                                              uint64_t lists, int l) {
    uint32_t hits = 0;
    uint64_t zeros = 0;
    while (lists) {
        __amdgpu_buffer_rsrc_t src[TCF_LISTS];
        int32_t n[TCF_LISTS], most = 0;
#pragma unroll
        for (int q = 0; q < TCF_LISTS; ++q) {
            const int k = lists ? __builtin_ctzll(lists) : 0;
            const uint64_t at = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(ys >> 32), k) << 32 |
                                (uint32_t)__builtin_amdgcn_readlane((int)ys, k);
            n[q] = lists ? __builtin_amdgcn_readlane(len, k) : 0;
            src[q] = __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t *>(ocol + at), 0, 4 * n[q], 0x00027000);
            most = max(most, n[q]);
            lists &= lists - 1;
        }
        for (int32_t j0 = 0; j0 < most; j0 += TCF_LOADS * WAVE) {
            uint32_t v[TCF_LISTS][TCF_LOADS];
#pragma unroll
            for (int q = 0; q < TCF_LISTS; ++q)
#pragma unroll
                for (int u = 0; u < TCF_LOADS; ++u)
                    v[q][u] = __builtin_amdgcn_raw_buffer_load_b32(src[q], 4 * (j0 + l) + 4 * u * WAVE, 0, 0);
#pragma unroll
            for (int q = 0; q < TCF_LISTS; ++q)
#pragma unroll
                for (int u = 0; u < TCF_LOADS; ++u) {
                    if (j0 + u * WAVE >= n[q]) continue;
                    hits += ((uint32_t)sx[v[q][u] >> 5] >> (v[q][u] & 31)) & 1u;
                    zeros += max(0, j0 + (u + 1) * WAVE - n[q]);
                }
        }
    }
    return (uint64_t)hits - (l == 0 && (sx[0] & 1) ? zeros : 0);
}

template <bool BITS>
__global__ __launch_bounds__(256) void k_tc_forward(int32_t n, const int64_t *__restrict__ ob,
                                                    const int64_t *__restrict__ oe,
                                                    const int32_t *__restrict__ ocol,
                                                    unsigned long long *total) {
    __shared__ __align__(8) int32_t s_nx[256 / WAVE][TCF_CAP];
    const int64_t wave_global = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / WAVE;
    const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) / WAVE;
    const int l = lane_id();
    int32_t *sx = s_nx[threadIdx.x / WAVE];
    uint64_t acc = 0;
    // the copy leaves the last words of the first wave's LDS to the block's sum (with more
    // LDS than 16 KB fewer blocks share a CU)
    unsigned long long *s_sum = reinterpret_cast<unsigned long long *>(&s_nx[0][TCF_CAP - 4]);
    int32_t *s_ended = &s_nx[0][TCF_CAP - 2];
    if (BITS) {
        for (int j = l; j < TCF_CAP; j += WAVE) sx[j] = 0;
        wave_sync();
    } else {
        if (threadIdx.x < 4) s_nx[0][TCF_CAP - 4 + threadIdx.x] = 0;
        __syncthreads();
    }
    for (int64_t x = wave_global; x < n; x += nwaves) {
        const int64_t xs = ob[x], xe = oe[x];
        const int64_t dx = xe - xs;
        if (dx < 2) continue;
        const bool staged = BITS || dx <= TCF_CAP - 4;
        int64_t tail = xe;  // BITS: the first entry with an id of TCF_IDS or more
        if (BITS) {
            int64_t small = 0;
            for (int64_t j0 = 0; j0 < dx; j0 += WAVE) {
                const int32_t v = j0 + l < dx ? ocol[xs + j0 + l] : TCF_IDS;
                if (v < TCF_IDS) atomicOr(&sx[v >> 5], (int32_t)(1u << (v & 31)));
                small += __popcll(ballot(v < TCF_IDS));
            }
            tail = xs + small;
            wave_sync();
        } else if (staged) {
            for (int64_t j = l; j < dx; j += WAVE) sx[j] = ocol[xs + j];
            wave_sync();
        }
        const auto in_bits = [&](int32_t v) {
            if (v < TCF_IDS) return ((uint32_t)sx[v >> 5] >> (v & 31) & 1u) != 0;
            return tail < xe && find_sorted(ocol, tail, xe, (uint32_t)v) >= 0;
        };
        const int64_t rx = (dx + WAVE - 1) / WAVE;
        for (int64_t p0 = 0; p0 < dx; p0 += WAVE) {
            // lane k fetches the list bounds of the k-th y of this chunk of N+(x)
            int64_t mys = 0, mye = 0;
            if (p0 + l < dx) {
                const int32_t y = !BITS && staged ? sx[p0 + l] : ocol[xs + p0 + l];
                mys = ob[y];
                mye = oe[y];
            }
            uint64_t rest = ballot(mye > mys);
            if (BITS) {
                const int32_t last = mye > mys ? ocol[mye - 1] : TCF_IDS;
                uint64_t low = ballot(last < TCF_IDS && mye - mys <= TCF_LONG * rx * WAVE);
                rest &= ~low;
                acc += bits_hits(sx, ocol, mys, (int32_t)(mye - mys), low, l);
            }
            const int cnt = (int)(dx - p0 < WAVE ? dx - p0 : WAVE);
            for (int k = 0; BITS ? rest != 0 : k < cnt; ++k) {
                if (BITS) {
                    k = __builtin_ctzll(rest);
                    rest &= rest - 1;
                }
                const int64_t ys = __shfl(mys, k, WAVE), ye = __shfl(mye, k, WAVE);
                const int64_t dy = ye - ys;
                if (staged && (dy + WAVE - 1) / WAVE <= 4 * rx) {
                    // four loads in flight per lane before the LDS searches
                    for (int64_t j0 = ys + l; j0 < ye; j0 += 4 * WAVE) {
                        int32_t v[4];
#pragma unroll
                        for (int u = 0; u < 4; ++u) v[u] = j0 + u * WAVE < ye ? ocol[j0 + u * WAVE] : -1;
#pragma unroll
                        for (int u = 0; u < 4; ++u)
                            if (v[u] >= 0 && (BITS ? in_bits(v[u]) : lds_has(sx, (int)dx, v[u]))) ++acc;
                    }
                } else {
                    for (int64_t j = xs + l; j < xe; j += WAVE)
                        if (find_sorted(ocol, ys, ye, (uint32_t)ocol[j]) >= 0) ++acc;
                }
            }
        }
        if (staged) wave_sync();  // the next row overwrites the staging
        if (BITS) {
            for (int64_t j = xs + l; j < tail; j += WAVE) sx[ocol[j] >> 5] = 0;
            wave_sync();
        }
    }
    // one add per block: a wave's add to the one total costs about 12 ns of a serial
    // chain (262k rows, 131k waves: 2.19 ms with an add per wave)
    acc = wave_sum(acc);
    if (BITS) {
        __shared__ uint64_t s_acc[256 / WAVE];
        if (l == 0) s_acc[threadIdx.x / WAVE] = acc;
        __syncthreads();
        if (threadIdx.x == 0) {
            for (int q = 1; q < 256 / WAVE; ++q) acc += s_acc[q];
            if (acc) atomicAdd(total, (unsigned long long)acc);
        }
    } else if (l == 0) {
        // the last wave to end adds; waves that end before it do not wait in their slots
        // (a barrier here: R-MAT 20 in the order given 74.1 ms, without 67.9)
        atomicAdd(s_sum, (unsigned long long)acc);
        wave_sync();
        if (atomicAdd(s_ended, 1) == 256 / WAVE - 1) {
            const unsigned long long all = atomicAdd(s_sum, 0ull);
            if (all) atomicAdd(total, all);
        }
    }
}

int tc_count_static(dg_graph *g, uint64_t *count) {
    DG_TRY(graph_merge(g));
    hipStream_t s = g->stream;
    Dir &F = g->fwd;
    const int32_t n = g->n;
    DG_TRY(g->ws.scan64.ensure((size_t)n + 1));
    const int blocks = (int)std::min<int64_t>(((int64_t)n + 3) / 4, 32768);
    // the forward list of x: entries ob[x] to oe[x] of ocol
    const int64_t *ob = F.off.p, *oe = g->ws.scan64.p;
    const int32_t *ocol = F.col.p;
    bool ordered = false, bits = false;
    if (g->relabeled) {
        DG_TRY(counters_clear(g));
        hipLaunchKernelGGL(k_tc_prefix, dim3(grid_wide(n)), dim3(WIDE_T), 0, s, n, F.off.p, F.col.p, F.deg.p, TCF_IDS,
                           g->ws.scan64.p, g->ws.dcnt + C_TC0, g->ws.dcnt + C_AUX0);
        DG_HIP(hipGetLastError());
        DG_TRY(counters_read(g));
        ordered = g->ws.hcnt[C_TC0] == 0;
        // (out of order the built lists differ, but batches change few of their entries)
        bits = (double)g->ws.hcnt[C_AUX0] >= TCF_LOW * (double)(F.m / 2);
    }
    if (!ordered) {
        // the merge's spare target buffers hold the oriented lists (m / 2 entries)
        DG_TRY(F.off2.ensure((size_t)n + 1));
        DG_TRY(F.col2.ensure((size_t)(F.m / 2) + 1));
        int64_t *odeg = g->ws.scan64.p;
        hipLaunchKernelGGL(k_tc_orient<false>, dim3(blocks), dim3(256), 0, s, n, F.off.p, F.col.p, F.deg.p, odeg,
                           nullptr, nullptr);
        DG_TRY(fill_i64(odeg + n, 0, 1, s));
        DG_TRY(scan_excl(g, odeg, F.off2.p, (int64_t)n + 1));
        hipLaunchKernelGGL(k_tc_orient<true>, dim3(blocks), dim3(256), 0, s, n, F.off.p, F.col.p, F.deg.p, nullptr,
                           F.off2.p, F.col2.p);
        ob = F.off2.p;
        oe = F.off2.p + 1;
        ocol = F.col2.p;
    }
    DG_TRY(counters_clear(g));
    unsigned long long *acc = reinterpret_cast<unsigned long long *>(g->ws.dcnt + C_TC1);
    hipLaunchKernelGGL(bits ? k_tc_forward<true> : k_tc_forward<false>,
                       dim3(std::min(blocks, bits ? TCF_BLOCKS : TCF_BLOCKS_COPY)), dim3(256), 0, s, n, ob, oe, ocol,
                       acc);
    DG_HIP(hipGetLastError());
    DG_TRY(counters_read(g));
    *count = (uint64_t)g->ws.hcnt[C_TC1];
    return DG_OK;
}

}  // namespace dg
