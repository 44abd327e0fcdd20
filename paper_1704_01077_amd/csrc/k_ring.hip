// Ring engine: searches on undirected graphs of low degree (street networks:
// high diameter), one per workgroup with its visited set in LDS; complete
// ones for the level-based updates (Sect. 7), cut ones for BFSCut (Sect. 6).
//
// Such a search is a thin ring that moves out over hundreds of levels.  The
// batched engine pays a grid barrier and several trips to memory for every
// one of those levels; here a level is separated by one workgroup barrier
// and its chain is queue -> row -> arc -> LDS bit, all inside one compute
// unit.  A visited bitmap of n bits fits the 160 KB of LDS up to about 1.2 M
// vertices, so every compute unit runs a search of its own and no arc costs
// an atomic outside LDS.
//
// A finished search leaves its vertices in level order in its queue; the
// workgroup then raises the bound of each of them (four queue positions a
// thread, their levels found in the level offsets by binary search) with an
// atomic maximum, which is sound in any order because
// every value written is a valid lower bound.  Numerators share one
// denominator per component ((r - 1)^2, exact for undirected graphs), so one
// 64-bit maximum updates a bound.
//
// What bounds it: on small graphs the latency of that chain (under 2 us a level
// on a grid of 2 10^4 vertices), on large ones cache lines from beyond the L2
// (on a grid of 10^6 3,576 searches expand 3.6 10^9 vertices in 60 ms, about one
// 128 B line each, the rate at which random lines reach the chip being 55 G/s).
// Measured against the batched engine, top 10 by NBBound: 27.4 -> 1.9 ms and
// 460 -> 60 ms.
#include <algorithm>

#include "dev_common.hpp"
#include "engine.hpp"

// threads of a workgroup (512 measured the same, 256 lost 19 % on 2 10^4 vertices)
#define RING_T 1024
// results a workgroup may hold back while the top k's lock is taken
#define RING_PEND 8
// vertices of a level kept in LDS beside the queue, levels whose offsets are
#define RING_FRONT 1024
#define RING_LEVELS 512

struct RingArgs {
    DevGraph g;
    DevReach rc;
    OrderView ov;
    BoundsView bv;
    DevTopk tk;
    RingWork w;
    int64_t* stats;
    int32_t words;
    int32_t lb_mode;
    int32_t limit;   // searches of this launch (0: no limit)
    int32_t gate;    // positions handed out before the top k is full
};

// The bound of a vertex is num / (r - 1)^2; Lev(l) - deg(w) is compared with
// num, so the engine keeps comb = num + deg and compares Lev(l) alone: one
// gather per vertex instead of two.  Deg bounds start as 0 / 1, and any other
// denominator than (r - 1)^2 falls back to the bound 0.  ell holds every
// vertex's first arcs in one 16-byte record (-1: none; more than four arcs:
// three, then -2 - the position of the fourth), so a search touches one
// cache line per vertex where row pointer and arcs took two (150 -> 82 ms of
// search time on a grid of 10^6 vertices).
__global__ void k_ring_begin(int32_t n, const int64_t* __restrict__ omega, const int32_t* __restrict__ deg,
                             const int64_t* __restrict__ num, const int64_t* __restrict__ den, int64_t* comb,
                             uint32_t* dec, const int32_t* __restrict__ rp, const int32_t* __restrict__ ci,
                             int4* __restrict__ ell, int32_t* cursor, int32_t from) {
    const int32_t v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= n) return;
    if (v == 0) *cursor = from;
    const int32_t b = rp[v], dv = rp[v + 1] - b;
    int4 r{-1, -1, -1, -1};
    if (dv > 0) r.x = ci[b];
    if (dv > 1) r.y = ci[b + 1];
    if (dv > 2) r.z = ci[b + 2];
    if (dv == 4) r.w = ci[b + 3];
    else if (dv > 4) r.w = -2 - (b + 3);
    ell[v] = r;
    const int64_t d = den[v], want = sq64(omega[v] - 1);
    comb[v] = deg[v] + (d == want ? num[v] : 0);
    if ((v & 31) == 0) dec[v >> 5] = 0;
}
__global__ void k_ring_end(int32_t n, const int64_t* __restrict__ omega, const int32_t* __restrict__ deg,
                           const int64_t* __restrict__ comb, int64_t* num, int64_t* den) {
    const int32_t v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= n || omega[v] <= 1) return;
    num[v] = comb[v] - deg[v];
    den[v] = sq64(omega[v] - 1);
}

// Marks the targets w (negative: none) of one pass in the LDS bitmap, each
// new one by exactly one thread, and appends those to the queue at out[...]
// and to the LDS copy of the next level (as far as that reaches), in the
// order of one LDS counter.
TKC_DEV void ring_visit(const int32_t (&w)[4], uint32_t* bits, int32_t spare, int32_t* out, int32_t* front,
                        int32_t* tail, uint64_t below) {
    // the four words are read together (no target: the spare word, which is
    // read but never marked: lanes that mark one word take turns)
    uint32_t word[4];
#pragma unroll
    for (int j = 0; j < 4; j++)
        word[j] = __hip_atomic_load(&bits[w[j] >= 0 ? w[j] >> 5 : spare], __ATOMIC_RELAXED,
                                    __HIP_MEMORY_SCOPE_WORKGROUP);
    bool isnew[4];
#pragma unroll
    for (int j = 0; j < 4; j++) {
        const uint32_t bit = 1u << (w[j] & 31);
        isnew[j] = w[j] >= 0 && !(word[j] & bit);
        if (isnew[j]) word[j] = for_wg(&bits[w[j] >> 5], bit);
    }
#pragma unroll
    for (int j = 0; j < 4; j++) isnew[j] = isnew[j] && !((word[j] >> (w[j] & 31)) & 1u);
    uint64_t m[4];
    int32_t c = 0;
#pragma unroll
    for (int j = 0; j < 4; j++) {
        m[j] = __ballot(isnew[j]);
        c += __popcll(m[j]);
    }
    if (c == 0) return;
    // the first active lane adds for all: the compiler may run the wave's
    // lanes through here in groups
    const int lane = lane_id();
    int32_t at = 0;
    if (lane == __builtin_amdgcn_readfirstlane(lane)) at = atomicAdd(tail, c);
    at = __builtin_amdgcn_readfirstlane(at);
#pragma unroll
    for (int j = 0; j < 4; j++) {
        if (isnew[j]) {
            const int32_t i = at + __popcll(m[j] & below);
            out[i] = w[j];
            front[i < RING_FRONT ? i : RING_FRONT] = w[j];   // the slot behind takes the rest
        }
        at += __popcll(m[j]);
    }
}

// Expands the frontier vertices base + thread: one aligned 16-byte load
// brings a vertex's first four arcs (ell); the few vertices with more go on
// through their rows.  cur is the LDS copy of the level or its part of the
// queue.  (Two or four vertices per thread and pass, or four threads per
// vertex, measured the same: the waves of a compute unit hide each other's
// latency.)
template <int T>
TKC_DEV void ring_expand(const RingArgs& a, uint32_t* bits, const int32_t* cur, int32_t items, int32_t base,
                         int32_t* out, int32_t* front, int32_t* tail, uint64_t below, int64_t& arcs) {
    const int32_t i = base + (int32_t)threadIdx.x;
    const int32_t u = i < items ? cur[i] : -1;
    int4 r{-1, -1, -1, -1};
    if (u >= 0) r = a.w.ell[u];
    int32_t w[4] = {r.x, r.y, r.z, r.w};
    int32_t b = 0, e = 0;
    if (w[3] < -1) {   // -2 - position of the fourth arc
        b = -2 - w[3];
        e = a.g.rp[u + 1];
        w[3] = -1;
    }
    arcs += (w[0] >= 0) + (w[1] >= 0) + (w[2] >= 0) + (w[3] >= 0) + (e - b);
    ring_visit(w, bits, a.words, out, front, tail, below);
    while (__any(b < e)) {
#pragma unroll
        for (int j = 0; j < 4; j++) w[j] = b + j < e ? a.g.ci[b + j] : -1;
        b += 4;
        ring_visit(w, bits, a.words, out, front, tail, below);
    }
}

// workgroup barrier that waits for this wave's LDS operations only: global
// stores (the queue, the level offsets) stay in flight
TKC_DEV void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

template <int T>
__global__ void __launch_bounds__(T) k_ring(RingArgs a) {
    extern __shared__ uint32_t s_bits[];
    __shared__ int32_t s_tail[3];
    __shared__ uint64_t s_mask[T / 64], s_omask[T / 64];
    __shared__ int32_t s_front[2][RING_FRONT + 1];
    __shared__ int32_t s_off[RING_LEVELS];
    __shared__ int64_t s_w64[T / 64];
    __shared__ int64_t s_x[3];
    __shared__ int64_t s_lim[2];
    __shared__ int32_t s_limid[2];
    __shared__ int64_t s_pS[RING_PEND], s_pR[RING_PEND], s_thr;
    __shared__ int32_t s_pI[RING_PEND];
    __shared__ int32_t s_pos, s_dec, s_cur;

    const int tid = threadIdx.x;
    const int lane = lane_id();
    const int wv = tid >> 6;
    const int32_t n = a.g.n;
    const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    const int32_t* __restrict__ deg = a.g.deg;
    int32_t* q = a.w.queue + (int64_t)blockIdx.x * RING_QSTRIDE(n);
    int32_t* off = a.w.levoff + (int64_t)blockIdx.x * a.w.lcap;
    int64_t* lev = a.w.levtab + (int64_t)blockIdx.x * a.w.lcap;
    const int32_t count = a.ov.count;
    int64_t st_mvis = 0, st_started = 0, st_exact = 0, st_cut = 0, st_skip = 0, st_maxl = 0, st_bytes = 0;

    for (int32_t i = tid; i < a.words; i += T) s_bits[i] = 0;
    // Alg. 1's tests of one position: 1 stop, 2 skip, 3 reaches nothing, 0 search
    auto judge = [&](int32_t p, const XVal& x) -> int {
        const int32_t v = a.ov.ord[p];
        const uint32_t key = a.ov.key[p];
        if (a.ov.key_is_bound ? key_stops(key, x) : (key == 0xffffffffu && x.den != 0)) return 1;
        const int64_t om = a.rc.omega[v];
        const int64_t num = ld_rlx(&a.w.comb[v]) - deg[v];
        if (lex_after(num, om <= 1 ? 0 : sq64(om - 1), TKC_OID(a.g, v), x.num, x.den, x.id)) return 2;
        return om <= 1 ? 3 : 0;
    };
    // Results wait in LDS until the top k's lock is free (first wave, which
    // also places them: one lane moving a list of 100 entries made 32 requests
    // on small street networks take 30 ms of 276): hundreds
    // of searches end at about the same time, and a workgroup that spun for
    // its turn would hold its compute unit and slow the lock's owner.  What
    // the top k would refuse by now leaves first (in all-ties mode x carries
    // the largest id, so that cannot tie with the k-th).
    int32_t npend = 0;
    auto offer = [&](bool wait) {   // called by the first wave's 64 lanes
        while (npend > 0) {
            const XVal x = read_x_poll(a.tk.st, a.tk.ring);
            const int64_t pS = s_pS[lane & (RING_PEND - 1)], pR = s_pR[lane & (RING_PEND - 1)];
            const int32_t pI = s_pI[lane & (RING_PEND - 1)];
            const bool stay = lane < npend && !lex_after(pS, pR <= 1 ? 0 : sq64(pR - 1), pI, x.num, x.den, x.id);
            uint64_t m = __ballot(stay);
            if (m) {
                int32_t got = 0;
                if (lane == 0) got = topk_try_lock(a.tk.st) ? 1 : 0;
                if (__shfl(got, 0, 64)) {
                    for (; m; m &= m - 1) {
                        const int l = __ffsll((long long)m) - 1;
                        topk_insert_wave_locked(a.tk.st, a.tk.ring, a.tk.S, a.tk.R, a.tk.I, shfl64(pS, l),
                                                shfl64(pR, l), __shfl(pI, l, 64));
                    }
                    if (lane == 0) topk_unlock(a.tk.st);
                } else {
                    __builtin_amdgcn_wave_barrier();
                    if (stay) {
                        const int32_t i = __popcll(m & below);
                        s_pS[i] = pS;
                        s_pR[i] = pR;
                        s_pI[i] = pI;
                    }
                    __builtin_amdgcn_wave_barrier();
                }
            }
            npend = __popcll(m);
            if (!wait) return;
            if (npend) __builtin_amdgcn_s_sleep(64);
        }
    };
    auto pend = [&](int64_t S, int64_t r, int32_t id) {
        if (lane == 0) {
            s_pS[npend] = S;
            s_pR[npend] = r;
            s_pI[npend] = id;
        }
        __builtin_amdgcn_wave_barrier();
        npend++;
        offer(npend == RING_PEND);
    };
    // the numerator over bden up to which a value does not pass x (exact when
    // x has that denominator: *id then breaks a tie, else none is cut on one)
    auto x_limit = [&](const XVal& x, int64_t bden, int32_t* id) -> int64_t {
        *id = 0x7fffffff;
        if (x.den == 0) return INT64_MAX - HEAVY_DEG;
        if (x.den == bden) {
            *id = x.id;
            return x.num;
        }
        const double t = (double)x.num * ((double)bden / (double)x.den) * (1.0 + 1e-9) + 2.0;
        return t < 9e18 ? (int64_t)t : INT64_MAX - HEAVY_DEG;
    };

    bool open = false;   // no waiting at the gate any more
    for (;;) {
        // ---- the next candidate: one position from the shared cursor; if it
        // is skipped, T positions at a time are judged and the cursor moves
        // past the skipped ones and the first that is not (compare-and-swap,
        // so no workgroup holds positions it is not working on; when another
        // was faster, the judged window serves for the next try)
        if (wv == 0) {
            // Until the top k is full nothing is cut or skipped, and where the
            // first searches fill it and end the order, others that started
            // meanwhile were in vain.  Positions from the gate on wait for those
            // before it, which are at least k, all in work, and never wait
            // themselves; a workgroup whose searches run deep does not wait (all
            // take long there, and it costs 2 % to say so to the others).
            // (Top 100 of trees of 3,000 and 150,000 vertices 1.80 -> 1.30 and 3.46
            // -> 2.06 ms with 256 searches for 2,000 and 1,000; top 1,000 18.8 ->
            // 7.1 and 16.8 -> 9.0.)
            int32_t p = -2, d = 4;   // 4: no more work for this workgroup
            for (;;) {
                offer(false);
                if (p == -2) {
                    p = -1;
                    if (lane == 0 && ld_rlx(a.w.stop) == 0 && (a.limit == 0 || ld_rlx(a.w.started) < a.limit))
                        p = fadd_rlx(a.w.cursor, 1);
                    p = __builtin_amdgcn_readfirstlane(p);
                }
                if (open || p < a.gate || p >= count) break;
                open = __builtin_amdgcn_readfirstlane(ld_rlx(&a.tk.st->seq) >= 0 ? 1 : 0);
                if (!open) __builtin_amdgcn_s_sleep(16);
            }
            if (lane == 0) {
                if (p >= 0 && p < count) {
                    d = judge(p, read_x_poll(a.tk.st, a.tk.ring));
                    st_skip += d == 2;
                }
                s_pos = p;
                s_dec = d;
            }
        }
        __syncthreads();
        int dec = s_dec;
        while (dec == 2) {
            __syncthreads();
            if (tid == 0) {
                s_cur = ld_rlx(a.w.cursor);
                const XVal x = read_x_poll(a.tk.st, a.tk.ring);
                s_x[0] = x.num; s_x[1] = x.den; s_x[2] = x.id;
            }
            __syncthreads();
            const int32_t c = s_cur;
            if (c >= count) { dec = 4; break; }   // uniform
            const XVal x{s_x[0], s_x[1], (int32_t)s_x[2]};
            const int d = c + tid < count ? judge(c + tid, x) : 2;
            const uint64_t m = __ballot(d != 2), mo = __ballot(d == 1 || d == 3);
            if (lane == 0) {
                s_mask[wv] = m;
                s_omask[wv] = mo;
            }
            __syncthreads();
            if (tid == 0) {
                const int32_t lim = count - c < T ? count - c : T;
                int32_t at = 0;   // the cursor, relative to the window
                s_dec = 2;
                while (at < lim) {
                    int32_t f = lim;
                    for (int w = at >> 6; w < T / 64; w++) {
                        const uint64_t mm = w == at >> 6 ? s_mask[w] & (~0ull << (at & 63)) : s_mask[w];
                        if (mm) { f = w * 64 + __ffsll((long long)mm) - 1; break; }
                    }
                    int32_t seen = c + at;
                    if (__hip_atomic_compare_exchange_strong(a.w.cursor, &seen, c + (f < lim ? f + 1 : lim),
                                                             __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                             __HIP_MEMORY_SCOPE_AGENT)) {
                        st_skip += f - at;
                        s_pos = c + f;
                        if (f < lim) s_dec = (s_omask[f >> 6] >> (f & 63)) & 1 ? judge(c + f, x) : 0;
                        break;
                    }
                    at = seen - c;
                }
            }
            __syncthreads();
            dec = s_dec;
        }
        if (dec == 4) break;
        const int32_t pos = s_pos;
        if (dec == 1) {
            if (tid == 0) for_rlx(a.w.stop, 1);
            break;
        }
        const int32_t v = a.ov.ord[pos];
        if (dec == 3) {
            if (tid == 0) {
                st_started++;
                st_exact++;
            }
            if (wv == 0) pend(0, 1, TKC_OID(a.g, v));
            __syncthreads();
            continue;
        }
        // ---- the search
        const int64_t rv = a.rc.omega[v], bden = sq64(rv - 1);   // undirected: r(v) is known
        const int32_t vid = TKC_OID(a.g, v);
        if (tid == 0) {
            if (a.limit) fadd_rlx(a.w.started, 1);
            s_bits[v >> 5] |= 1u << (v & 31);
            q[0] = v;
            s_front[0][0] = v;
            off[0] = 0;
            s_off[0] = 0;
            s_tail[0] = 0;
            s_tail[1] = 0;
            s_tail[2] = 0;
        }
        __syncthreads();
        // level D holds q[ls, le); level D + 1 is appended at q[le ...) through
        // the counter of parity D % 3, which is cleared one level ahead
        int32_t D = 0, ls = 0, le = 1;
        int64_t SD = 0;
        bool cut = false;
        for (;;) {
            const int c3 = D % 3;
            // BFSCut with the levels up to D known exactly: every other vertex
            // is at least D + 1 away (at least what Lemma 6.1 gives at level
            // D - 1, whose bound on the size of level D is now its size).  x
            // is polled by the last wave at every fourth level, into the slot
            // that is not read until the next poll
            const bool cuts = a.lb_mode == 0 || (a.lb_mode == 2 && D <= CUTLB_DEPTH);
            if (cuts && D > 0) {
                const int sl = ((D - 1) >> 2) & 1;
                const int64_t bound = SD + (int64_t)(D + 1) * (rv - le);
                if (bound > s_lim[sl] || (bound == s_lim[sl] && vid > s_limid[sl])) { cut = true; break; }
            }
            if (cuts && (D & 3) == 0 && tid == T - 64) {
                int32_t id;
                s_lim[(D >> 2) & 1] = x_limit(read_x_poll(a.tk.st, a.tk.ring), bden, &id);
                s_limid[(D >> 2) & 1] = id;
            }
            if (tid == 0) {
                const int nx = D % 3 == 2 ? 0 : c3 + 1;
                s_tail[nx] = 0;
                if (D + 1 < a.w.lcap) off[D + 1] = le;
                if (D + 1 < RING_LEVELS) s_off[D + 1] = le;
            }
            const int32_t items = le - ls;
            int32_t* front = s_front[(D + 1) & 1];
            if (items <= RING_FRONT) {
                for (int32_t b = 0; b < items; b += T)
                    ring_expand<T>(a, s_bits, s_front[D & 1], items, b, q + le, front, &s_tail[c3], below, st_mvis);
            } else {
                for (int32_t b = 0; b < items; b += T)
                    ring_expand<T>(a, s_bits, q + ls, items, b, q + le, front, &s_tail[c3], below, st_mvis);
            }
            lds_barrier();
            const int32_t cnt = s_tail[c3];
            D++;
            SD += (int64_t)D * cnt;
            ls = le;
            le += cnt;
            if (cnt == 0) break;
            // a level wider than its LDS copy is read from the queue
            if (cnt > RING_FRONT) __syncthreads();
        }
        // complete: D - 1 is the last level, q[0, le) the vertices in level
        // order, off[l] the start of level l for l <= D
        __syncthreads();   // the queue and the offsets are written
        const int32_t r = le;
        const int32_t maxD = D - 1;
        open |= D > TKC_DEEP;
        if (tid == 0) {
            st_started++;
            const int64_t md = cut ? D : maxD;
            if (md > st_maxl) st_maxl = md;
            st_bytes += 12 * (int64_t)le;
            if (cut) st_cut++;
            else st_exact++;
        }
        if (wv == 0 && !cut) {
            pend(SD, r, vid);
            // a bound above the limit is above x: no later search need raise it
            int32_t id;
            const int64_t lim = a.lb_mode ? x_limit(read_x_poll(a.tk.st, a.tk.ring), bden, &id) : 0;
            if (lane == 0) s_thr = lim;
        }
        // the bitmap has done its work: it takes the bits of the vertices whose
        // bound needs no update, all of one pass's tests then stay in LDS
        const bool update = a.lb_mode != 0 && !cut && maxD >= 1 && D + 1 < a.w.lcap;
        for (int32_t i = tid; i < a.words; i += T) s_bits[i] = update ? ld_rlx(&a.w.dec[i]) : 0;
        if (!update) {
            // deeper than the level tables: no update, and the batched engine
            // takes the rest of the order
            if (a.lb_mode != 0 && !cut && maxD >= 1 && tid == 0) for_rlx(a.w.stop, 2);
        } else {
            // Lev(l) for l >= 1 (off[D] = r closes the table): Lev(1) from the
            // sums, then prefix sums of the steps
            // low_l - (r - pre_l), low_l = vertices at level <= l - 3,
            // pre_l = vertices at level <= l + 1
            int64_t run = SD - r + 1 + 2 * (int64_t)(off[2 <= D ? 2 : D] - off[1]) +
                          (maxD >= 2 ? (int64_t)(off[3] - off[2]) : 0);
            if (tid == 0) lev[1] = run;
            for (int32_t b = 2; b <= maxD; b += T) {
                const int32_t l = b + tid;
                int64_t step = 0;
                if (l <= maxD)
                    step = (l >= 3 ? (int64_t)off[l - 2] : 0) - ((int64_t)r - off[l + 2 <= D ? l + 2 : D]);
                int64_t inc = step;
#pragma unroll
                for (int o = 1; o < 64; o <<= 1) {
                    const int64_t y = __shfl_up(inc, o, 64);
                    if (lane >= o) inc += y;
                }
                if (lane == 63) s_w64[wv] = inc;
                __syncthreads();
                int64_t before = run, all = run;
                for (int w = 0; w < T / 64; w++) {
                    if (w < wv) before += s_w64[w];
                    all += s_w64[w];
                }
                if (l <= maxD) lev[l] = before + inc;
                run = all;
                __syncthreads();
            }
            __syncthreads();
            const int64_t thr = s_thr + HEAVY_DEG;
            const int32_t* lo_off = D < RING_LEVELS ? s_off : off;
            // (a vertex raised above thr is taken off by who raised it; one
            // that was above already, by the workgroups its word falls to:
            // hundreds of searches pass over the same words)
            for (int32_t i0 = 4 * tid; i0 < r; i0 += 4 * T) {
                const int4 w4 = *(const int4*)(q + i0);   // q is 16-byte aligned and has room
                const int32_t w[4] = {w4.x, w4.y, w4.z, w4.w};
                bool todo[4], any = false;
#pragma unroll
                for (int j = 0; j < 4; j++) {
                    todo[j] = i0 + j > 0 && i0 + j < r;
                    todo[j] = todo[j] && !((s_bits[todo[j] ? w[j] >> 5 : 0] >> (w[j] & 31)) & 1u);
                    any |= todo[j];
                }
                if (!any) continue;
                // cached copies of the bounds may be old, never too high
                int64_t cc[4];
#pragma unroll
                for (int j = 0; j < 4; j++) cc[j] = todo[j] ? a.w.comb[w[j]] : 0;
                // level: the last whose first position is not behind i
                int32_t lo = 1, hi = D;
                while (hi - lo > 1) {
                    const int32_t mid = (lo + hi) >> 1;
                    if (lo_off[mid] <= i0) lo = mid; else hi = mid;
                }
#pragma unroll
                for (int j = 0; j < 4; j++) {
                    while (lo + 1 < D && lo_off[lo + 1] <= i0 + j) lo++;
                    if (!todo[j]) continue;
                    const uint32_t bit = 1u << (w[j] & 31);
                    const int64_t L = lev[lo];
                    int64_t c = cc[j];
                    if (L > c) c = ld_rlx(&a.w.comb[w[j]]);
                    if (L > c) {
                        __hip_atomic_fetch_max(&a.w.comb[w[j]], L, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        if (L > thr) for_rlx(&a.w.dec[w[j] >> 5], bit);
                    } else if (c > thr && (((w[j] >> 5) ^ (int32_t)blockIdx.x) & 31) == 0) {
                        for_rlx(&a.w.dec[w[j] >> 5], bit);
                    }
                }
            }
            __syncthreads();
            for (int32_t i = tid; i < a.words; i += T) s_bits[i] = 0;
        }
        __syncthreads();
    }
    if (wv == 0) offer(true);
    st_mvis = wave_sum_i64(st_mvis);
    if (lane == 0 && st_mvis) {
        fadd_rlx(&a.stats[ST_MVIS], st_mvis);
        fadd_rlx(&a.stats[ST_BYTES], 4 * st_mvis);
    }
    if (tid == 0) {
        int64_t* s = a.stats;
        if (st_started) fadd_rlx(&s[ST_STARTED], st_started);
        if (st_exact) fadd_rlx(&s[ST_EXACT], st_exact);
        if (st_cut) fadd_rlx(&s[ST_CUT], st_cut);
        if (st_skip) fadd_rlx(&s[ST_SKIPPED], st_skip);
        if (st_bytes) fadd_rlx(&s[ST_BYTES], st_bytes);
        __hip_atomic_fetch_max(&s[ST_MAXLEVEL], st_maxl, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// the kernels' static LDS: two level copies, the offsets, and under 1 KiB more
#define RING_STATIC_LDS (4 * (2 * RING_FRONT + RING_LEVELS) + 1024)

// the bitmap and a spare word
static size_t ring_lds_bytes(int32_t n) { return 4 * (((size_t)n + 31) / 32 + 1); }

// Undirected, so that every r(v) is known; no heavy vertex, since one lane
// expands a vertex; few arcs, or a level would be wide and few in number and
// the batched engine's shared reads pay.  Up to that line the ring is ahead at
// low diameter too: batched -> ring, top 10 by NBCut of sparse random graphs
// of 3 10^4 vertices, 4 arcs a vertex 3.8 -> 1.3 ms, 7 arcs 11.7 -> 2.0 ms; of
// 3 10^5, 35 -> 11.7 and 74 -> 26 ms; a small world of 3 10^4, 131 -> 5.6 ms.
// (Large shallow graphs fill the top k batched: tkc_ring_seeds.)
int tkc_ring_blocks(const DevGraph& g) {
    if (g.directed || g.nheavy > 0 || g.m > 8 * (int64_t)g.n || g.n < 2) return 0;
    if (ring_lds_bytes(g.n) + RING_STATIC_LDS > (size_t)tkc_lds_limit()) return 0;
    const int cus = tkc_cu_count();
    return cus > 0 ? cus : 0;
}

// A complete search of one workgroup takes 4.7 ms on a tree of 10^6 vertices,
// 64 of them batched half of that, and they often end the query: top 10 by
// NBCut and NBBound 7.1 -> 4.2 and 9.1 -> 4.9 ms, of a random graph of 7 10^6
// arcs, top 1, 17.2 -> 6.4; trees of 3 10^5 2.5 -> 2.0 and 3.0 -> 2.3, of 1.5 10^5
// 1.7 -> 1.5, but a random graph of as many vertices and 4.5 10^5 arcs 3.3 -> 3.6.
// On a deep graph a batch pays a grid barrier for every one of its levels.
bool tkc_ring_seeds(const DevGraph& g, int32_t levels) { return levels <= TKC_DEEP && g.n > (1 << 18); }

int tkc_launch_ring_begin(const DevGraph& g, const DevReach& rc, const BoundsView& bv, const RingWork& w,
                          int32_t from, hipStream_t s) {
    hipLaunchKernelGGL(k_ring_begin, dim3((g.n + 255) / 256), dim3(256), 0, s, g.n, rc.omega, (const int32_t*)g.deg,
                       (const int64_t*)bv.num, (const int64_t*)bv.den, w.comb, w.dec, g.rp, g.ci, w.ell, w.cursor, from);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}
int tkc_launch_ring_end(const DevGraph& g, const DevReach& rc, const BoundsView& bv, const RingWork& w, hipStream_t s) {
    hipLaunchKernelGGL(k_ring_end, dim3((g.n + 255) / 256), dim3(256), 0, s, g.n, rc.omega, (const int32_t*)g.deg,
                       (const int64_t*)w.comb, bv.num, bv.den);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int tkc_launch_ring(const DevGraph& g, DevReach rc, OrderView ov, BoundsView bv, DevTopk tk, RingWork w,
                    int64_t* stats, int lb_mode, int32_t k, int32_t limit, hipStream_t s) {
    if (!w.queue || !w.levoff || !w.levtab || !w.comb || !w.dec || !w.ell || !w.cursor || !w.stop || !w.started || w.nblocks < 1 || w.lcap < 4)
        return -2;
    if (g.directed || g.nheavy > 0 || bv.harm) return -2;
    const size_t lds = ring_lds_bytes(g.n);
    if (lds + RING_STATIC_LDS > (size_t)tkc_lds_limit()) return -2;
    RingArgs a{};
    a.g = g; a.rc = rc; a.ov = ov; a.bv = bv; a.tk = tk; a.w = w;
    a.stats = stats;
    a.words = (int32_t)(lds / 4) - 1;
    a.lb_mode = lb_mode;
    a.limit = limit;
    a.gate = std::max(k, w.nblocks);
    const void* fn = (const void*)k_ring<RING_T>;
    if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess) hipGetLastError();
    hipLaunchKernelGGL(k_ring<RING_T>, dim3(w.nblocks), dim3(RING_T), lds, s, a);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}
