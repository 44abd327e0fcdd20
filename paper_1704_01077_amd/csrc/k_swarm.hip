// Per-workgroup engine: most BFSCut searches of Alg. 1 stop after two or
// three levels (Sect. 6), far too little work to fill the GPU one search at
// a time.  Here every workgroup pulls the next candidate from the order
// with an atomic cursor and runs that search alone: levels are separated by
// workgroup barriers only, the visited set is a bitmap in LDS, the queue is
// private, and the current k-th farness x is polled at every level boundary.  A search whose
// queue outgrows its capacity is handed back (deferred) to the batched
// engine, which is better at large searches.  The stop rule of Alg. 1 is
// applied when a candidate is taken: once one candidate's key proves that
// every later bound exceeds x, the cursor is closed for all workgroups.
//
// Deferred searches do not lower x, so on a graph where most candidates
// reach a large part of the graph quickly the workgroups would walk the
// whole order deferring everything.  After `defer_cap` deferrals the engine
// therefore closes itself: the cursor stops, searches in flight are
// deferred at their next level boundary, and the host hands the deferred
// list and the rest of the order to the batched engine.
//
// What bounds it: the latency of a level (cursor, row, arc, bitmap, barrier),
// so the bitmap lives in LDS (in memory, with the polls of x invalidating the
// L2 at every level, the traversal of a social network of 3 10^4 vertices, top
// 100, took 1.71 ms and of a web graph of 3 10^4, top 10, 0.37; now 0.72 and
// 0.28).  A large search wants the whole chip, and a batch shares its reads
// among 64 of them.  Up to TKC_SWARM_SIZE this engine follows the batched seeds
// at once; batched -> this engine, social networks of 3 10^4 vertices and 1.8
// 10^5 edges 2.34 -> 0.72 ms, web graphs of 3 10^4 and 1.8 10^5 0.89 -> 0.54
// (top 100).  Beyond, it depends on the graph (web graphs of 6 10^4 and 4.8 10^5
// 1.28 -> 2.24, of 1.5 10^5 and 1.3 10^6 1.90 -> 4.27, others the other way), and
// a few batches behind the seeds show which (tkc_swarm_pays).
//
// stop word bits: 1 = the stop rule fired, 2 = the engine closed itself.
#include "dev_common.hpp"
#include "engine.hpp"

#include <stdlib.h>

// workgroup size: big enough that one search keeps many arcs in flight
// (the searches left after the seed batch are few and large on complex
// networks); TKC_SWARM_SB=256 or 1024 picks one for experiments
#define SB_DEFAULT 1024
static int swarm_sb() {
    static const int v = [] {
        const char* e = getenv("TKC_SWARM_SB");
        const int x = e ? atoi(e) : SB_DEFAULT;
        return x == 256 ? 256 : (x == 1024 ? 1024 : SB_DEFAULT);
    }();
    return v;
}

struct SwarmArgs {
    DevGraph g;
    DevReach rc;
    OrderView ov;
    BoundsView bv;
    DevTopk tk;
    SwarmWork w;
    int64_t* stats;
    int32_t start_pos;
    int32_t words;        // of the bitmap: the dynamic LDS
    int32_t defer_cap;
};

// exclusive scan of one int per thread over the workgroup; returns the total
template <int SB>
TKC_DEV int32_t block_excl_scan(int32_t v, int32_t* out, int32_t* wsum) {
    int32_t x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        int32_t y = __shfl_up(x, o, 64);
        if (lane_id() >= o) x += y;
    }
    int wv = threadIdx.x >> 6;
    if (lane_id() == 63) wsum[wv] = x;
    __syncthreads();
    int32_t base = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < SB / 64; w++) {
        int32_t t = wsum[w];
        if (w < wv) base += t;
        tot += t;
    }
    *out = base + x - v;
    return tot;
}

template <int SB>
__global__ void __launch_bounds__(SB) k_swarm(SwarmArgs a) {
    extern __shared__ uint32_t s_vis[];
    __shared__ int32_t s_pos;
    __shared__ int32_t s_pre[SB + 1];
    __shared__ int32_t s_beg[SB];
    __shared__ int32_t s_wsum[SB / 64];
    __shared__ int32_t s_tail;
    __shared__ int32_t s_over;
    __shared__ int64_t s_cnt, s_deg;
    __shared__ int64_t s_x[3];
    __shared__ int32_t s_dec;
    __shared__ int32_t s_closed;

    const int tid = threadIdx.x;
    const int32_t* __restrict__ rp = a.g.rp;
    const int32_t* __restrict__ ci = a.g.ci;
    const int32_t* __restrict__ deg = a.g.deg;
    const bool dir = a.g.directed;
    int32_t* q = a.w.queue + (int64_t)blockIdx.x * a.w.qcap;
    const int32_t qcap = a.w.qcap;
    const int32_t count = a.ov.count;
    int64_t st_mvis = 0, st_started = 0, st_exact = 0, st_cut = 0, st_skip = 0, st_def = 0;
    int64_t st_maxl = 0, st_bytes = 0;
    // the preceding batch (same stream, finished) hands over where it stopped
    int32_t start_pos = a.start_pos;
    bool seed_stopped = false;
    if (a.w.seed) {
        start_pos = (int32_t)a.w.seed[ST_CURSOR];
        seed_stopped = a.w.seed[ST_STOP] != 0;
    }

    for (int32_t i = tid; i < a.words; i += SB) s_vis[i] = 0;
    for (;;) {
        if (tid == 0) {
            int32_t p = -1;
            if (!seed_stopped && ld_rlx(a.w.stop) == 0) p = start_pos + fadd_rlx(a.w.cursor, 1);
            s_pos = p;
            const XVal x = read_x_poll(a.tk.st, a.tk.ring);
            s_x[0] = x.num; s_x[1] = x.den; s_x[2] = x.id;
            s_dec = 0;
            if (p >= 0 && p < count) {
                int32_t v = a.ov.ord[p];
                uint32_t key = a.ov.key[p];
                bool stop = a.bv.harm ? key_stops_h(key, x)
                                      : (a.ov.key_is_bound ? key_stops(key, x) : (key == 0xffffffffu && x.den != 0));
                if (stop) { for_rlx(a.w.stop, 1); s_dec = 1; }
                else if (lex_after(a.bv.num[v], a.bv.den[v], TKC_OID(a.g, v), x.num, x.den, x.id)) { s_dec = 2; st_skip++; }
                else if (a.rc.omega[v] <= 1) {
                    s_dec = 3;
                    st_started++; st_exact++;
                    if (a.bv.harm) topk_insert(a.tk.st, a.tk.ring, a.tk.S, a.tk.R, a.tk.I, harm_enc(0.0), 2, TKC_OID(a.g, v));
                    else topk_insert(a.tk.st, a.tk.ring, a.tk.S, a.tk.R, a.tk.I, 0, 1, TKC_OID(a.g, v));
                }
            } else {
                s_dec = 1;
            }
        }
        __syncthreads();
        const int32_t pos = s_pos;
        const int dec = s_dec;
        __syncthreads();
        if (dec == 1) break;
        if (dec != 0) continue;

        const int32_t v = a.ov.ord[pos];
        const int64_t av = a.rc.alpha[v], ov = a.rc.omega[v];
        const int64_t dv = deg[v];
        if (tid == 0) {
            s_vis[v >> 5] |= 1u << (v & 31);
            q[0] = v;
            s_tail = 1;
            s_over = 0;
        }
        __syncthreads();
        int64_t D = 0, nD = 1, SD = 0, U = dv, nf = 1;
        double H = 0.0;   // harmonic centrality so far (levels 1..D)
        int32_t ls = 0, le = 1;
        int status = 0;   // 1 exact, 2 cut, 3 deferred
        int64_t mvis = 0;
        for (;;) {
            if (nf == 0) { status = 1; break; }
            if (tid == 0) {
                const XVal x = read_x_poll(a.tk.st, a.tk.ring);
                s_x[0] = x.num; s_x[1] = x.den; s_x[2] = x.id;
                s_cnt = 0; s_deg = 0;
                s_closed = (ld_rlx(a.w.stop) & 2) != 0;
            }
            __syncthreads();
            {
                int64_t bn, bd;
                if (a.bv.harm) harm_cut_bound(H, nD, U, D, ov, &bn, &bd);
                else cut_bound(SD, nD, U, D, av, ov, &bn, &bd);
                if (lex_after(bn, bd, TKC_OID(a.g, v), s_x[0], s_x[1], (int32_t)s_x[2])) { status = 2; break; }
            }
            if (s_closed) { status = 3; break; }
            // expand level D: frontier q[ls, le), edge-balanced in chunks of SB vertices
            int64_t my_cnt = 0, my_deg = 0;
            for (int32_t c = ls; c < le; c += SB) {
                int32_t i = c + tid;
                int32_t d = 0, b = 0;
                if (i < le) {
                    int32_t u = q[i];
                    b = rp[u];
                    d = rp[u + 1] - b;
                }
                int32_t pre;
                int32_t tot = block_excl_scan<SB>(d, &pre, s_wsum);
                s_pre[tid] = pre;
                s_beg[tid] = b;
                if (tid == 0) s_pre[SB] = tot;
                __syncthreads();
                mvis += tot;
                for (int32_t e = tid; e < tot; e += SB) {
                    // owner: last j with s_pre[j] <= e
                    int32_t lo = 0, hi = SB;
                    while (hi - lo > 1) {
                        int32_t mid = (lo + hi) >> 1;
                        if (s_pre[mid] <= e) lo = mid; else hi = mid;
                    }
                    int32_t w = ci[s_beg[lo] + (e - s_pre[lo])];
                    uint32_t bit = 1u << (w & 31);
                    if (!(s_vis[w >> 5] & bit)) {
                        const uint32_t old = atomicOr(&s_vis[w >> 5], bit);
                        if (!(old & bit)) {
                            int32_t slot = atomicAdd(&s_tail, 1);
                            if (slot < qcap) q[slot] = w;
                            else s_over = 1;
                            my_cnt++;
                            my_deg += deg[w];
                        }
                    }
                }
                __syncthreads();
            }
            my_cnt = wave_sum_i64(my_cnt);
            my_deg = wave_sum_i64(my_deg);
            if (lane_id() == 0 && my_cnt) {
                atomicAdd((unsigned long long*)&s_cnt, (unsigned long long)my_cnt);
                atomicAdd((unsigned long long*)&s_deg, (unsigned long long)my_deg);
            }
            __syncthreads();
            if (s_over) { status = 3; break; }
            int64_t cnt = s_cnt, dsum = s_deg;
            D++;
            nD += cnt;
            SD += D * cnt;
            if (a.bv.harm) H += (double)cnt / (double)D;
            U = dir ? dsum : dsum - cnt;
            nf = cnt;
            ls = le;
            le = s_tail;
            __syncthreads();
        }
        // clear the bitmap: by the queue where that is shorter and did not
        // overflow (then some marked vertices are not in it)
        if (s_tail < a.words && s_tail <= qcap) {
            const int32_t tail = s_tail;
            for (int32_t i = tid; i < tail; i += SB) s_vis[q[i] >> 5] = 0;
        } else {
            for (int32_t i = tid; i < a.words; i += SB) s_vis[i] = 0;
        }
        if (status == 1 && tid < 64) {
            if (a.bv.harm) topk_insert_wave(a.tk.st, a.tk.ring, a.tk.S, a.tk.R, a.tk.I, harm_enc(H), 2, TKC_OID(a.g, v));
            else topk_insert_wave(a.tk.st, a.tk.ring, a.tk.S, a.tk.R, a.tk.I, SD, nD, TKC_OID(a.g, v));
        }
        if (tid == 0) {
            st_started++;
            st_mvis += mvis;
            st_bytes += 8 * mvis + 12 * (int64_t)le + 16 * (nD - 1);
            int64_t md = status == 1 ? D - 1 : D;
            if (md > st_maxl) st_maxl = md;
            if (status == 1) {
                st_exact++;
            } else if (status == 2) {
                st_cut++;
            } else {
                st_def++;
                st_started--;
                // every candidate is taken once, so slot < n
                int32_t slot = fadd_rlx(a.w.ndeferred, 1);
                a.w.deferred[slot] = v;
                if (slot + 1 >= a.defer_cap) for_rlx(a.w.stop, 2);
            }
        }
        __syncthreads();
    }
    if (tid == 0) {
        int64_t* s = a.stats;
        if (st_mvis) fadd_rlx(&s[ST_MVIS], st_mvis);
        if (st_started) fadd_rlx(&s[ST_STARTED], st_started);
        if (st_exact) fadd_rlx(&s[ST_EXACT], st_exact);
        if (st_cut) fadd_rlx(&s[ST_CUT], st_cut);
        if (st_skip) fadd_rlx(&s[ST_SKIPPED], st_skip);
        if (st_def) fadd_rlx(&s[ST_DEFERRED], st_def);
        if (st_bytes) fadd_rlx(&s[ST_BYTES], st_bytes);
        __hip_atomic_fetch_max(&s[ST_MAXLEVEL], st_maxl, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

bool tkc_swarm_small(const DevGraph& g) {
    return g.n + (g.directed ? (int64_t)g.m : (int64_t)g.m / 2) <= TKC_SWARM_SIZE;
}
// the kernel's static LDS: rows and their prefix sums, and under 1 KiB more
#define SWARM_STATIC_LDS (8 * 1024 + 1024)
static size_t swarm_lds_bytes(int32_t n) { return 4 * (((size_t)n + 31) / 32); }
// A level costs a batch a grid barrier, 7 us shared by 64 searches, and this
// engine some workgroup barriers; an arc costs a batch its share of one read
// of the frontier's rows, and this engine 1 / 150 ns of the whole chip.
// Batched -> this engine, us a search, by arcs and levels: random graphs of 4
// 10^4 vertices (28,000, 6) 1.33 -> 0.40; of 2 10^4 (11,900, 3) 0.85 -> 0.14;
// of 6 10^4 and 3 10^6 arcs (126,000, 4) 1.41 -> 0.75; small worlds of 6.2 10^4
// (44,000, 22) 2.86 -> 0.46, (105,000, 95) 9.34 -> 1.32; a king's lattice of one-way
// streets of 6.25 10^4, 142 levels, 12.9 -> 1.5; but web graphs of 6 10^4 and 3.8
// 10^6 arcs (812,000, 4) 1.18 -> 3.52, a social network of 2 10^4 and 8 10^5
// (178,000, 3) 1.09 -> 2.89.
bool tkc_swarm_pays(double arcs, int64_t levels) { return arcs <= (1 << 17) + 8192.0 * (double)levels; }
bool tkc_swarm_fits(const DevGraph& g) {
    return swarm_lds_bytes(g.n) + SWARM_STATIC_LDS <= (size_t)tkc_lds_limit();
}

// Plain mode on a small graph: this engine with one workgroup takes the same
// searches in the same order (same counters), and a level costs it a few
// workgroup barriers where the grid of the plain engine pays three grid
// barriers.  Whole queries, top 10: social networks of 2,000 vertices and 2 10^4
// edges 8.5 -> 2.0 ms, web graphs of 4,000 and 4 10^4 arcs 39.6 -> 7.3, of 8,000
// and 8 10^4 43 -> 13; the line lies where the whole chip begins to pay for
// complete searches (16,000 and 1.6 10^5, top 1: 1.16 -> 1.79).
bool tkc_plain_small(const DevGraph& g) { return g.n + (int64_t)g.m <= (1 << 17); }
// A complete search takes this engine about 0.9 ns an arc, the plain engine some 75
// us whatever the graph's size here: those that fill the top k go to the faster.
// Social networks of 2,000 vertices and 1.2 10^5 arcs, top 10, 1.32 -> 0.84 ms, web
// graphs of 5,000 and 10^5 arcs 1.79 -> 1.37; of 1,000 and 5.5 10^4 0.82 here
// against 0.97 by the plain engine.
bool tkc_plain_first(const DevGraph& g) { return g.n + (int64_t)g.m > (1 << 16); }

int tkc_swarm_max_blocks(int block) {
    (void)block;
    const int cus = tkc_cu_count();
    if (cus < 1) return -1;
    int occ = 0;
    const int sb = swarm_sb();
    if (sb == 1024) {
        occ = tkc_occupancy((const void*)k_swarm<1024>, 1024);
        if (occ < 0) return -1;
        if (occ > 2) occ = 2;
    } else {
        occ = tkc_occupancy((const void*)k_swarm<256>, 256);
        if (occ < 0) return -1;
        if (occ > 8) occ = 8;
    }
    return cus * (occ > 0 ? occ : 1);
}

int tkc_launch_swarm(const DevGraph& g, DevReach rc, OrderView ov, BoundsView bv, DevTopk tk,
                     SwarmWork w, int64_t* stats, int32_t start_pos, const EngineTuning& tune,
                     hipStream_t s) {
    (void)tune;
    SwarmArgs a{};
    a.g = g; a.rc = rc; a.ov = ov; a.bv = bv; a.tk = tk; a.w = w;
    a.stats = stats;
    a.start_pos = start_pos;
    if (!tkc_swarm_fits(g)) return -2;
    const size_t lds = swarm_lds_bytes(g.n);
    a.words = (int32_t)(lds / 4);
    const void* fn = swarm_sb() == 1024 ? (const void*)k_swarm<1024> : (const void*)k_swarm<256>;
    if (lds > (32 << 10) &&
        hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
        hipGetLastError();
    a.defer_cap = w.defer_cap > 0 ? w.defer_cap : 0x7fffffff;
    if (swarm_sb() == 1024)
        hipLaunchKernelGGL(k_swarm<1024>, dim3(w.nblocks), dim3(1024), lds, s, a);
    else
        hipLaunchKernelGGL(k_swarm<256>, dim3(w.nblocks), dim3(256), lds, s, a);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}
