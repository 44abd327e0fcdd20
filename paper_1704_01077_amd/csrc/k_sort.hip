// Stable LSD radix sort of (uint32 key, int32 value) pairs, 8-bit digits: the
// processing order of Alg. 1 (values start as vertex ids, so equal keys keep
// ascending ids) and the arcs between components.  Digits on which all keys
// agree are skipped.
// A tile is RS8_TILE items taken round-robin (item j * 256 + t is thread t's
// j-th), so rounds in order and lanes in order visit the tile in order.
// Per pass: per-tile digit counts; per digit, the exclusive prefix over
// tiles and the total; the scatter, which ranks each round's items by
// digit within each wave (a match over the digit's eight bits) and keeps
// running per-digit counts in LDS.  (4-bit digits take two launches a pass
// instead of three but twice the passes: 80 against 57 us of kernels for 17
// varying bits of 10^5 keys.)
#include "dev_common.hpp"
#include "engine.hpp"

__global__ void k_rs_mask(const uint32_t* __restrict__ keys, int32_t n, uint32_t* mask) {
    // mask[0] = OR of keys, mask[1] = OR of their complements, both from 0
    uint32_t o = 0, a = 0xffffffffu;
    const int32_t t0 = blockIdx.x * blockDim.x + threadIdx.x, step = gridDim.x * blockDim.x;
    int32_t head = 0;
    if (((uintptr_t)keys & 15u) == 0) {
        // 16-byte loads, independent across the loop
        const uint4* k4 = (const uint4*)keys;
        head = n & ~3;
        for (int32_t i = t0; i < head / 4; i += step) {
            const uint4 q = k4[i];
            o |= q.x | q.y | q.z | q.w;
            a &= q.x & q.y & q.z & q.w;
        }
    }
    for (int32_t i = head + t0; i < n; i += step) {
        const uint32_t k = keys[i];
        o |= k; a &= k;
    }
#pragma unroll
    for (int s = 32; s > 0; s >>= 1) {
        o |= __shfl_xor(o, s, 64);
        a &= __shfl_xor(a, s, 64);
    }
    __shared__ uint32_t so[4], sa[4];
    if (lane_id() == 0) { so[threadIdx.x >> 6] = o; sa[threadIdx.x >> 6] = a; }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < (int)(blockDim.x >> 6); w++) { o |= so[w]; a &= sa[w]; }
        __hip_atomic_fetch_or(&mask[0], o, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_fetch_or(&mask[1], ~a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

#define RS8_THREADS 256
#define RS8_ROUNDS 8
#define RS8_TILE (RS8_THREADS * RS8_ROUNDS)

static inline int rs8_tiles(int32_t n) { return (n + RS8_TILE - 1) / RS8_TILE; }

TKC_DEV uint64_t below_lanes() {
    const int l = lane_id();
    return l == 0 ? 0ull : (~0ull >> (64 - l));
}

// lanes of the wave whose (valid) digit equals this lane's; all 64 lanes call
TKC_DEV uint64_t rs8_match(uint32_t d, bool valid) {
    uint64_t m = __ballot(valid);
#pragma unroll
    for (int b = 0; b < 8; b++) {
        const uint64_t bal = __ballot((d >> b) & 1u);
        m &= ((d >> b) & 1u) ? bal : ~bal;
    }
    return m;
}

// cnt[d * tiles + tile] = items of digit d in the tile
__global__ void __launch_bounds__(RS8_THREADS) k_rs8_count(const uint32_t* __restrict__ keys, int32_t n, int shift,
                                                            int32_t* cnt, int32_t tiles) {
    __shared__ int32_t h[256];
    const int t = threadIdx.x;
    h[t] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * RS8_TILE;
#pragma unroll
    for (int j = 0; j < RS8_ROUNDS; j++) {
        const int64_t i = base + j * RS8_THREADS + t;
        const bool valid = i < n;
        const uint32_t d = valid ? (keys[i] >> shift) & 255u : 0u;
        const uint64_t m = rs8_match(d, valid);
        if (valid && __ffsll((long long)m) - 1 == lane_id()) atomicAdd(&h[d], __popcll(m));
    }
    __syncthreads();
    cnt[(int64_t)t * tiles + blockIdx.x] = h[t];
}

// workgroup d: the exclusive prefix of digit d's counts over the tiles, in
// place, and the digit's total
__global__ void __launch_bounds__(RS8_THREADS) k_rs8_scan(int32_t* cnt, int32_t tiles, int32_t* total) {
    __shared__ int32_t wsum[RS8_THREADS / 64];
    int32_t* row = cnt + (int64_t)blockIdx.x * tiles;
    const int t = threadIdx.x;
    const int32_t per = (tiles + RS8_THREADS - 1) / RS8_THREADS;
    const int32_t lo = t * per, hi = lo + per < tiles ? lo + per : tiles;
    int32_t s = 0;
    for (int32_t q = lo; q < hi; q++) s += row[q];
    int32_t x = s;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int32_t y = __shfl_up(x, o, 64);
        if (lane_id() >= o) x += y;
    }
    if (lane_id() == 63) wsum[t >> 6] = x;
    __syncthreads();
    int32_t run = x - s;
    for (int w = 0; w < (t >> 6); w++) run += wsum[w];
    for (int32_t q = lo; q < hi; q++) {
        const int32_t c = row[q];
        row[q] = run;
        run += c;
    }
    if (t == RS8_THREADS - 1) total[blockIdx.x] = run;
}

__global__ void __launch_bounds__(RS8_THREADS) k_rs8_scatter(const uint32_t* __restrict__ keys,
                                                              const int32_t* __restrict__ vals, int32_t n, int shift,
                                                              const int32_t* __restrict__ pre, int32_t tiles,
                                                              const int32_t* __restrict__ total,
                                                              uint32_t* __restrict__ okeys, int32_t* __restrict__ ovals) {
    __shared__ int32_t start[256];   // where digit d's items of this tile go
    __shared__ int32_t run[256];     // of which this many are placed
    __shared__ int32_t wc[RS8_THREADS / 64][256];
    __shared__ int32_t wsum[RS8_THREADS / 64];
    const int t = threadIdx.x, wv = t >> 6, lane = lane_id();
    {   // digits before d over the whole input, then this tile's prefix in d
        const int32_t tot = total[t];
        int32_t x = tot;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int32_t y = __shfl_up(x, o, 64);
            if (lane >= o) x += y;
        }
        if (lane == 63) wsum[wv] = x;
        __syncthreads();
        int32_t below = x - tot;
        for (int w = 0; w < wv; w++) below += wsum[w];
        start[t] = below + pre[(int64_t)t * tiles + blockIdx.x];
        run[t] = 0;
    }
    const int64_t base = (int64_t)blockIdx.x * RS8_TILE;
    for (int j = 0; j < RS8_ROUNDS; j++) {
        const int64_t i = base + j * RS8_THREADS + t;
        const bool valid = i < n;
        uint32_t k = 0;
        int32_t v = 0;
        if (valid) {
            k = keys[i];
            v = vals[i];
        }
        const uint32_t d = (k >> shift) & 255u;
#pragma unroll
        for (int w = 0; w < RS8_THREADS / 64; w++) wc[w][t] = 0;
        __syncthreads();
        const uint64_t m = rs8_match(d, valid);
        if (valid && __ffsll((long long)m) - 1 == lane) wc[wv][d] = __popcll(m);
        __syncthreads();
        if (valid) {
            int32_t pos = start[d] + run[d] + __popcll(m & below_lanes());
            for (int w = 0; w < wv; w++) pos += wc[w][d];
            okeys[pos] = k;
            ovals[pos] = v;
        }
        __syncthreads();
        int32_t add = 0;
#pragma unroll
        for (int w = 0; w < RS8_THREADS / 64; w++) add += wc[w][t];
        run[t] += add;
    }
}

// All of a small sort in one workgroup: every wave holds 256 consecutive items
// in registers, ranks them digit by digit as the scatter above does, and the
// workgroup trades them through LDS.  Seven launches and a host wait for the
// keys' mask, about 60 us, become one of 18 us at 2,000 keys.
#define RSS_MAX 4096
__global__ void __launch_bounds__(1024) k_rs_small(uint32_t* keys, int32_t* vals, int32_t n) {
    __shared__ uint32_t s_k[RSS_MAX];
    __shared__ int32_t s_v[RSS_MAX];
    __shared__ int32_t wc[16][256];
    __shared__ int32_t start[256], wsum[4];
    __shared__ uint32_t s_or, s_nor;
    const int t = threadIdx.x, wv = t >> 6, lane = lane_id();
    uint32_t k[4], o = 0, no = 0;
    int32_t v[4];
#pragma unroll
    for (int j = 0; j < 4; j++) {
        const int32_t i = wv * 256 + j * 64 + lane;
        k[j] = i < n ? keys[i] : 0u;
        v[j] = i < n ? vals[i] : 0;
        if (i < n) {
            o |= k[j];
            no |= ~k[j];
        }
    }
    if (t == 0) s_or = s_nor = 0;
    __syncthreads();
    atomicOr(&s_or, o);
    atomicOr(&s_nor, no);
    __syncthreads();
    const uint32_t vary = s_or & s_nor;
    for (int shift = 0; shift < 32; shift += 8) {
        if (((vary >> shift) & 255u) == 0) continue;
        for (int i = t; i < 16 * 256; i += 1024) wc[i >> 8][i & 255] = 0;
        __syncthreads();
        int32_t rank[4];
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const bool valid = wv * 256 + j * 64 + lane < n;
            const uint32_t d = (k[j] >> shift) & 255u;
            const uint64_t m = rs8_match(d, valid);
            const int32_t before = valid ? wc[wv][d] : 0;
            rank[j] = before + __popcll(m & below_lanes());
            __builtin_amdgcn_wave_barrier();
            if (valid && __ffsll((long long)m) - 1 == lane) wc[wv][d] = before + __popcll(m);
            __builtin_amdgcn_wave_barrier();
        }
        __syncthreads();
        int32_t run = 0, x = 0;
        if (t < 256) {
            for (int w = 0; w < 16; w++) {
                const int32_t c = wc[w][t];
                wc[w][t] = run;
                run += c;
            }
            x = run;
#pragma unroll
            for (int sh = 1; sh < 64; sh <<= 1) {
                const int32_t y = __shfl_up(x, sh, 64);
                if (lane >= sh) x += y;
            }
            if (lane == 63) wsum[wv] = x;
        }
        __syncthreads();
        if (t < 256) {
            for (int w = 0; w < wv; w++) x += wsum[w];
            start[t] = x - run;
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 4; j++)
            if (wv * 256 + j * 64 + lane < n) {
                const uint32_t d = (k[j] >> shift) & 255u;
                const int32_t p = start[d] + wc[wv][d] + rank[j];
                s_k[p] = k[j];
                s_v[p] = v[j];
            }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const int32_t i = wv * 256 + j * 64 + lane;
            k[j] = i < n ? s_k[i] : 0u;
            v[j] = i < n ? s_v[i] : 0;
        }
    }
#pragma unroll
    for (int j = 0; j < 4; j++) {
        const int32_t i = wv * 256 + j * 64 + lane;
        if (i < n) {
            keys[i] = k[j];
            vals[i] = v[j];
        }
    }
}

int64_t tkc_sort8_hist_words(int32_t n) { return 256LL * rs8_tiles(n > 0 ? n : 1) + 256 + 16; }

int tkc_sort_mask(const uint32_t* keys, int32_t n, uint32_t* mask_dev, uint32_t* mask_host, hipStream_t s) {
    if (n <= RSS_MAX) return 0;   // sorted without it
    if (hipMemsetAsync(mask_dev, 0, 2 * sizeof(uint32_t), s) != hipSuccess) return -1;
    int gb = rs8_tiles(n);
    if (gb > 256) gb = 256;
    hipLaunchKernelGGL(k_rs_mask, dim3(gb), dim3(256), 0, s, keys, n, mask_dev);
    if (hipMemcpyAsync(mask_host, mask_dev, 2 * sizeof(uint32_t), hipMemcpyDeviceToHost, s) != hipSuccess)
        return -1;
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int tkc_sort_pairs8(uint32_t* keys, int32_t* vals, uint32_t* tmp_keys, int32_t* tmp_vals, int32_t n, int32_t* hist,
                    uint32_t* mask_dev, uint32_t* mask_host, hipStream_t s, const uint32_t* known_mask) {
    if (n <= 1) return 0;
    if (n <= RSS_MAX) {
        hipLaunchKernelGGL(k_rs_small, dim3(1), dim3(1024), 0, s, keys, vals, n);
        return hipGetLastError() == hipSuccess ? 0 : -1;
    }
    if (!known_mask) {
        if (tkc_sort_mask(keys, n, mask_dev, mask_host, s)) return -1;
        if (hipStreamSynchronize(s) != hipSuccess) return -1;
        known_mask = mask_host;
    }
    const uint32_t vary = known_mask[0] & known_mask[1];
    const int tiles = rs8_tiles(n);
    int32_t* total = hist + 256LL * tiles;
    uint32_t* ka = keys; int32_t* va = vals;
    uint32_t* kb = tmp_keys; int32_t* vb = tmp_vals;
    for (int shift = 0; shift < 32; shift += 8) {
        if (((vary >> shift) & 255u) == 0) continue;
        hipLaunchKernelGGL(k_rs8_count, dim3(tiles), dim3(RS8_THREADS), 0, s, ka, n, shift, hist, tiles);
        hipLaunchKernelGGL(k_rs8_scan, dim3(256), dim3(RS8_THREADS), 0, s, hist, tiles, total);
        hipLaunchKernelGGL(k_rs8_scatter, dim3(tiles), dim3(RS8_THREADS), 0, s, ka, va, n, shift,
                           (const int32_t*)hist, tiles, (const int32_t*)total, kb, vb);
        uint32_t* tk = ka; ka = kb; kb = tk;
        int32_t* tv = va; va = vb; vb = tv;
    }
    if (ka != keys) {
        hipMemcpyAsync(keys, ka, sizeof(uint32_t) * (size_t)n, hipMemcpyDeviceToDevice, s);
        hipMemcpyAsync(vals, va, sizeof(int32_t) * (size_t)n, hipMemcpyDeviceToDevice, s);
    }
    return hipGetLastError() == hipSuccess ? 0 : -1;
}
