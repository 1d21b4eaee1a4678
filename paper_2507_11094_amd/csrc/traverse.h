// Frontier expansion shared by the traversals (SSSP push, subtree invalidation,
// decremental pull, PageRank reach closure).
//
// A wave takes up to 64 frontier vertices, scans their degrees (base row + diff
// row) with a 64-lane prefix sum and then walks the concatenated edge slots 256 at
// a time, EX_U per lane, so every lane always has an edge regardless of the degree
// mix (a load-balanced search inside the wave).  Vertices with more than
// `heavy_deg` edges are not expanded in place: they are cut into chunks of `chunk`
// edges that a second kernel spreads over the whole grid, one wave per chunk.
//
// The steps are bound by latency: an edge costs a chain of dependent accesses
// (neighbour id, its state, an atomic on it, its stamp), and the frontiers of most
// rounds do not fill the device.  So
//   - a lane issues each stage of the chain for EX_U slots before it waits for the
//     first, in place of one slot at a time;
//   - a short frontier is spread over more waves (expand_vpw vertices per wave): 64
//     adjacent hubs of the degree order are up to 32,768 edges for one wave;
//   - a block of four waves reserves its output once, because every add on the one
//     counter costs about 12 ns in series, and the traversal tally is spread over
//     TALLY_SLOTS cache lines.
#pragma once

#include <algorithm>

#include "dg_device.h"

namespace dg {

struct DirView {
    const int64_t *off;
    const int32_t *col;
    const int32_t *w;
    const int64_t *doff;
    const int32_t *dcol;
    const int32_t *dw;
};

inline DirView view(const Dir &d) { return DirView{d.off.p, d.col.p, d.w.p, d.doff.p, d.dcol.p, d.dw.p}; }

struct ExpandArgs {
    const int32_t *F;   // frontier
    int64_t nf;
    const int64_t *nfp = nullptr;  // when set, the frontier length is read from device memory
    DirView g;
    int64_t *hq;        // heavy chunk queue: (v << 32) | chunk
    int64_t *hcount;    // its length
    int heavy_deg;
    int chunk;
    // when set: the entries of the rows this step walks are added to the slots
    // tally[j * TALLY_STRIDE], j < TALLY_SLOTS (traversal tally)
    int64_t *tally = nullptr;
    int vpw = WAVE;     // frontier vertices per wave (a power of two; device counts: set in the kernel)
};

// Vertices per wave: 64, or fewer (down to 8) while that would leave fewer than
// 2,048 waves, eight per CU.  With 64 always, a 10,000-vertex frontier ran on 157
// waves.
constexpr int64_t EX_WAVES = 2048;
__host__ __device__ __forceinline__ int expand_vpw(int64_t nf) {
    int v = WAVE;
    while (v > 8 && nf < EX_WAVES * v) v >>= 1;
    return v;
}

// Output of an expansion: vertices the op selects go to `out` (and `out2`, when
// set) with their lengths in `count` / `count2`.  SPLIT ops choose one of the two
// lists per vertex instead (see the op interface).
struct SinkTarget {
    int32_t *out = nullptr;
    int64_t *count = nullptr;
    int32_t *out2 = nullptr;
    int64_t *count2 = nullptr;
};

// Threads per block of the expansion kernels.  They run beside the PageRank tiles: where
// five workgroups of these share a CU (hot rows), they leave 10 KB of LDS and 12 waves, and
// a block of four waves with 4 KB fits; where eight do, they hold every wave slot, and a
// block takes the place of a tile that ends.  A block of eight waves with 26 KB waited for
// several tiles to end (cut walk on R-MAT 22, beside six: 68 -> 172 us a level).
constexpr int EX_T = 256;
constexpr int EX_W = EX_T / WAVE;
constexpr int EX_U = 4;             // slots per lane in flight

// Per-wave staging of selected vertices in LDS: one atomic per WB_CAP entries while
// the wave walks, and one per block for what is left at its end (same-address
// atomics serialise).
constexpr int WB_CAP = 256;
struct WaveSink {
    int32_t *buf;
    int n;
    int32_t *out;
    int64_t *count;
    int32_t *out2;
    int64_t *count2;
    __device__ __forceinline__ void copy(int64_t b1, int64_t b2) {
        for (int j = lane_id(); j < n; j += WAVE) {
            const int32_t x = buf[j];
            out[b1 + j] = x;
            if (out2) out2[b2 + j] = x;
        }
    }
    __device__ __forceinline__ void flush() {
        wave_sync();
        int64_t b1 = 0, b2 = 0;
        if (lane_id() == 0) {
            b1 = (int64_t)atomicAdd((unsigned long long *)count, (unsigned long long)n);
            if (out2) b2 = (int64_t)atomicAdd((unsigned long long *)count2, (unsigned long long)n);
        }
        b1 = __shfl(b1, 0, WAVE);
        b2 = __shfl(b2, 0, WAVE);
        copy(b1, b2);
        wave_sync();
        n = 0;
    }
    __device__ __forceinline__ void push(bool p, int32_t x) {
        const uint64_t m = ballot(p);
        const int c = __popcll(m);
        if (c == 0) return;
        if (n + c > WB_CAP) flush();
        if (p) buf[n + __popcll(m & lanemask_lt())] = x;
        n += c;
    }
};

// What the waves of a block still hold goes out with one atomic per list (all
// threads of the block call this).
struct SinkShared {
    int n[EX_W];
    int64_t b1, b2;
};
__device__ __forceinline__ void sink_finish(WaveSink &k, SinkShared &sh) {
    const int wv = threadIdx.x / WAVE;
    if (lane_id() == 0) sh.n[wv] = k.n;
    __syncthreads();
    int before = 0, tot = 0;
#pragma unroll
    for (int q = 0; q < EX_W; ++q) {
        const int c = sh.n[q];
        if (q < wv) before += c;
        tot += c;
    }
    if (tot == 0) return;  // uniform
    if (threadIdx.x == 0) {
        sh.b1 = (int64_t)atomicAdd((unsigned long long *)k.count, (unsigned long long)tot);
        if (k.out2) sh.b2 = (int64_t)atomicAdd((unsigned long long *)k.count2, (unsigned long long)tot);
    }
    __syncthreads();
    k.copy(sh.b1 + before, k.out2 ? sh.b2 + before : 0);
}

// Op interface (every call is made by every lane of the wave in lock-step; valid
// marks real edges, and x is 0 where it is false):
//   static constexpr bool W        the op reads edge weights
//   static constexpr bool REDUCE   the op takes a minimum at the frontier vertex
//   static constexpr bool SPLIT    selected vertices go to one of two lists
//   bool vtx(int32_t v, int32_t &payload)     false: skip v
//   P peek(int32_t x)                          state of x, loaded ahead
//   REDUCE:  uint64_t cand(valid, payload, x, w, P)    ~0: nothing to offer
//            void commit(int32_t v, uint64_t c)        c: minimum over a run of v's edges
//   else:    T attempt(valid, v, payload, x, w, P)     first atomic of the chain
//            int select(valid, v, payload, x, w, T)    0: nothing, 1: x goes to the
//                 sink's list, 2 (SPLIT): to its second list
//   SinkTarget sink() const                    -- out == nullptr: no output
// EX_U slots of a lane: entry loads, then the op's stages one after the other.
// valid[u]: slot u holds an entry; cp / wp: its place; own[u]: number of its row
// in the wave (equal over a run of slots).
template <class Op, bool ONE_ROW>
__device__ __forceinline__ void expand_slots(const Op &op, WaveSink &sk, WaveSink &sk2, bool (&valid)[EX_U],
                                             const int32_t *const (&cp)[EX_U], const int32_t *const (&wp)[EX_U],
                                             const int32_t (&v)[EX_U], const int32_t (&pay)[EX_U],
                                             const int (&own)[EX_U]) {
    int32_t x[EX_U], wt[EX_U];
#pragma unroll
    for (int u = 0; u < EX_U; ++u) {
        x[u] = *cp[u];
        wt[u] = Op::W ? *wp[u] : 0;
    }
#pragma unroll
    for (int u = 0; u < EX_U; ++u) {
        valid[u] = valid[u] && !((uint32_t)x[u] & DEAD);
        x[u] = valid[u] ? (int32_t)((uint32_t)x[u] & ID_MASK) : 0;
    }
    decltype(op.peek(0)) pk[EX_U];
#pragma unroll
    for (int u = 0; u < EX_U; ++u) pk[u] = op.peek(x[u]);
    if constexpr (Op::REDUCE) {
        uint64_t c[EX_U];
#pragma unroll
        for (int u = 0; u < EX_U; ++u) c[u] = op.cand(valid[u], pay[u], x[u], wt[u], pk[u]);
        if constexpr (ONE_ROW) {
            uint64_t m = c[0];
#pragma unroll
            for (int u = 1; u < EX_U; ++u) m = c[u] < m ? c[u] : m;
            m = wave_min(m);
            if (lane_id() == 0 && m != ~0ull) op.commit(v[0], m);
        } else {
            // the first slot of each run gets the run's minimum within the 64 slots
            const int l = lane_id();
#pragma unroll
            for (int u = 0; u < EX_U; ++u) {
                uint64_t m = c[u];
#pragma unroll
                for (int d = 1; d < WAVE; d <<= 1) {
                    const uint64_t y = __shfl_down(m, d, WAVE);
                    const int oo = __shfl_down(own[u], d, WAVE);
                    if (l + d < WAVE && oo == own[u] && y < m) m = y;
                }
                const int op1 = __shfl_up(own[u], 1, WAVE);
                if ((l == 0 || op1 != own[u]) && m != ~0ull) op.commit(v[u], m);
            }
        }
    } else {
        decltype(op.attempt(false, 0, 0, 0, 0, pk[0])) at[EX_U];
#pragma unroll
        for (int u = 0; u < EX_U; ++u) at[u] = op.attempt(valid[u], v[u], pay[u], x[u], wt[u], pk[u]);
        int sel[EX_U];
#pragma unroll
        for (int u = 0; u < EX_U; ++u) sel[u] = op.select(valid[u], v[u], pay[u], x[u], wt[u], at[u]);
        if (sk.out) {
#pragma unroll
            for (int u = 0; u < EX_U; ++u) {
                sk.push(sel[u] == 1, x[u]);
                if constexpr (Op::SPLIT) sk2.push(sel[u] == 2, x[u]);
            }
        }
    }
}

template <class Op>
__global__ __launch_bounds__(EX_T) void k_expand(ExpandArgs a, Op op) {
    __shared__ int32_t s_sink[Op::SPLIT ? 2 : 1][EX_W][WB_CAP];
    __shared__ SinkShared s_fin;
    const int wv = threadIdx.x / WAVE, l = lane_id();
    const SinkTarget t = op.sink();
    WaveSink sk{s_sink[0][wv], 0, t.out, t.count, Op::SPLIT ? nullptr : t.out2, t.count2};
    WaveSink sk2{s_sink[Op::SPLIT ? 1 : 0][wv], 0, t.out2, t.count2, nullptr, nullptr};
    const int64_t wave_global = (int64_t)blockIdx.x * EX_W + wv;
    const int64_t nwaves = (int64_t)gridDim.x * EX_W;
    const int64_t nf = a.nfp ? *a.nfp : a.nf;
    const int vpw = a.nfp ? expand_vpw(nf) : a.vpw;
    int64_t walked = 0;  // entries of this lane's rows (heavy rows too, walked by k_expand_heavy)
    for (int64_t wb = wave_global * vpw; wb < nf; wb += nwaves * vpw) {
        const int64_t fi = wb + l;
        int32_t v = -1, pay = 0;
        int64_t ob = 0, od = 0;
        int32_t db = 0, tot = 0;
        if (l < vpw && fi < nf) {
            v = a.F[fi];
            const int64_t o0 = a.g.off[v], o1 = a.g.off[v + 1], d0 = a.g.doff[v], d1 = a.g.doff[v + 1];
            if (op.vtx(v, pay)) {
                ob = o0;
                db = (int32_t)(o1 - o0);
                od = d0;
                tot = db + (int32_t)(d1 - d0);
            }
        }
        walked += tot;
        // split heavy vertices into grid-wide chunks
        const bool heavy = tot > a.heavy_deg;
        if (ballot(heavy)) {
            const int32_t nch = heavy ? (tot + a.chunk - 1) / a.chunk : 0;
            const int64_t incl_ch = wave_incl_scan((int64_t)nch);
            const int64_t tot_ch = __shfl(incl_ch, WAVE - 1, WAVE);
            int64_t base_ch = 0;
            if (l == 0) base_ch = atomicAdd((unsigned long long *)a.hcount, (unsigned long long)tot_ch);
            base_ch = __shfl(base_ch, 0, WAVE);
            for (int32_t c = 0; c < nch; ++c)
                a.hq[base_ch + incl_ch - nch + c] = ((int64_t)v << 32) | (uint32_t)c;
            if (heavy) tot = 0;
        }
        // load-balanced walk over the light vertices' edges (a wave's rows are
        // distinct, so its slots number fewer than 2^32)
        const uint32_t incl = wave_incl_scan((uint32_t)tot);
        const uint32_t excl = incl - (uint32_t)tot;
        const uint32_t T = (uint32_t)__shfl((int)incl, WAVE - 1, WAVE);
        const int64_t pb = ob - (int64_t)excl;       // base and diff position of slot 0
        const int64_t pd = od - (int64_t)excl - db;
        const uint32_t split = excl + (uint32_t)db;  // first slot of the row's diff entries
        const bool diffs = ballot(tot > db) != 0;    // uniform
        for (uint64_t eb = 0; eb < T; eb += WAVE * EX_U) {
            bool valid[EX_U];
            const int32_t *cp[EX_U], *wp[EX_U];
            int32_t vo[EX_U], po[EX_U];
            int own[EX_U];
            uint32_t e[EX_U];
#pragma unroll
            for (int u = 0; u < EX_U; ++u) {
                const uint64_t s = eb + (uint64_t)(u * WAVE + l);
                valid[u] = s < T;
                e[u] = (uint32_t)s;
                own[u] = 0;
            }
#pragma unroll
            for (int step = 32; step > 0; step >>= 1) {
#pragma unroll
                for (int u = 0; u < EX_U; ++u) {
                    const uint32_t x = (uint32_t)__shfl((int)excl, own[u] + step, WAVE);
                    if (x <= e[u]) own[u] += step;
                }
            }
#pragma unroll
            for (int u = 0; u < EX_U; ++u) {
                const int o = own[u];
                vo[u] = __shfl(v, o, WAVE);
                po[u] = __shfl(pay, o, WAVE);
                // slots past the end read the frontier instead, so that no load
                // sits behind a branch that the wave would wait at
                const int64_t i = __shfl(pb, o, WAVE) + (int64_t)e[u];
                cp[u] = valid[u] ? a.g.col + i : a.F;
                wp[u] = valid[u] ? a.g.w + i : a.F;
            }
            if (diffs) {
#pragma unroll
                for (int u = 0; u < EX_U; ++u) {
                    const int64_t i = __shfl(pd, own[u], WAVE) + (int64_t)e[u];
                    if ((uint32_t)__shfl((int)split, own[u], WAVE) <= e[u] && valid[u]) {
                        cp[u] = a.g.dcol + i;
                        wp[u] = a.g.dw + i;
                    }
                }
            }
            expand_slots<Op, false>(op, sk, sk2, valid, cp, wp, vo, po, own);
        }
    }
    if (sk.out) sink_finish(sk, s_fin);
    if constexpr (Op::SPLIT) {
        __syncthreads();
        sink_finish(sk2, s_fin);
    }
    if (a.tally) {  // uniform: one add per block
        __shared__ int64_t s_walked[EX_W];
        walked = wave_sum(walked);
        if (l == 0) s_walked[wv] = walked;
        __syncthreads();
        if (threadIdx.x == 0) {
            int64_t s = 0;
            for (int w = 0; w < EX_W; ++w) s += s_walked[w];
            if (s)
                atomicAdd((unsigned long long *)(a.tally + (blockIdx.x % TALLY_SLOTS) * TALLY_STRIDE),
                          (unsigned long long)s);
        }
    }
}

// One wave per heavy chunk (grid-stride over the queue).
template <class Op>
__global__ __launch_bounds__(EX_T) void k_expand_heavy(ExpandArgs a, Op op) {
    const int64_t nq = *a.hcount;
    if ((int64_t)blockIdx.x * EX_W >= nq) return;  // uniform
    __shared__ int32_t s_sink[Op::SPLIT ? 2 : 1][EX_W][WB_CAP];
    __shared__ SinkShared s_fin;
    const int wv = threadIdx.x / WAVE, l = lane_id();
    const SinkTarget t = op.sink();
    WaveSink sk{s_sink[0][wv], 0, t.out, t.count, Op::SPLIT ? nullptr : t.out2, t.count2};
    WaveSink sk2{s_sink[Op::SPLIT ? 1 : 0][wv], 0, t.out2, t.count2, nullptr, nullptr};
    const int64_t wave_global = (int64_t)blockIdx.x * EX_W + wv;
    const int64_t nwaves = (int64_t)gridDim.x * EX_W;
    for (int64_t qi = wave_global; qi < nq; qi += nwaves) {
        const int64_t ent = a.hq[qi];
        const int32_t v = (int32_t)(ent >> 32);
        const int32_t c = (int32_t)(ent & 0xffffffff);
        int32_t pay = 0;
        if (!op.vtx(v, pay)) continue;  // uniform across the wave
        const int64_t ob = a.g.off[v];
        const int32_t db = (int32_t)(a.g.off[v + 1] - ob);
        const int64_t od = a.g.doff[v];
        const int32_t tot = db + (int32_t)(a.g.doff[v + 1] - od);
        const int64_t s = (int64_t)c * a.chunk;
        const int64_t e = min((int64_t)tot, s + a.chunk);
        for (int64_t jb = s; jb < e; jb += WAVE * EX_U) {
            bool valid[EX_U];
            const int32_t *cp[EX_U], *wp[EX_U];
            int32_t vo[EX_U], po[EX_U];
            int own[EX_U];
#pragma unroll
            for (int u = 0; u < EX_U; ++u) {
                const int64_t j = jb + u * WAVE + l;
                valid[u] = j < e;
                const bool diff = j >= db;
                const int64_t i = diff ? od + (j - db) : ob + j;
                cp[u] = valid[u] ? (diff ? a.g.dcol : a.g.col) + i : a.F;
                wp[u] = valid[u] ? (diff ? a.g.dw : a.g.w) + i : a.F;
                vo[u] = v;
                po[u] = pay;
                own[u] = 0;
            }
            expand_slots<Op, true>(op, sk, sk2, valid, cp, wp, vo, po, own);
        }
    }
    if (sk.out) sink_finish(sk, s_fin);
    if constexpr (Op::SPLIT) {
        __syncthreads();
        sink_finish(sk2, s_fin);
    }
}

// Host side: run one expansion step of `op` over frontier F (nf entries).
// hcount must point at a zeroed device counter.  heavy_deg = NO_HEAVY: no row is
// cut into chunks (every row is walked by k_expand) and the chunk kernel is not
// launched.
constexpr int NO_HEAVY = 0x7fffffff;
constexpr int EX_BLOCKS = 2048;  // 32 waves per CU; longer frontiers are walked grid-stride
template <class Op>
inline int launch_expand(hipStream_t s, const ExpandArgs &args, const Op &op) {
    if (!args.nfp && args.nf <= 0) return DG_OK;
    ExpandArgs a = args;
    int64_t blocks = EX_BLOCKS;  // device-side count: fixed grid-stride grid
    if (!a.nfp) {
        a.vpw = expand_vpw(a.nf);
        blocks = std::min<int64_t>((a.nf + (int64_t)EX_W * a.vpw - 1) / ((int64_t)EX_W * a.vpw), EX_BLOCKS);
    }
    hipLaunchKernelGGL(k_expand<Op>, dim3((unsigned)blocks), dim3(EX_T), 0, s, a, op);
    if (a.heavy_deg != NO_HEAVY)
        hipLaunchKernelGGL(k_expand_heavy<Op>, dim3(EX_BLOCKS), dim3(EX_T), 0, s, a, op);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return set_error(DG_EDEVICE, "expand launch failed: %s", hipGetErrorString(e));
    return DG_OK;
}

}  // namespace dg
