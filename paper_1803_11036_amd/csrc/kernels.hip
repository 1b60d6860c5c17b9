// HIP kernels (gfx950, wave64) of the sliding super point detector.
//
// Cell encoding: a sliding-estimator cell is one byte.  0 = never hit; a hit
// in slot s stores the stamp 1 + (s mod 255).  At the close of slot t the
// cell's distance (Sec. 3.2 distance recorder) is (stamp(t) - stamp) mod 255,
// valid because every cell whose distance reaches k is cleared before it can
// reach 255 (rotating expiry, see k_hot_detect).  This replaces the paper's
// 16-bit recorder and its +1 sweep over all recorders every slot (Sec. 4.3)
// with one byte per cell and no per-slot write pass.
//
// Liveness test (distance < k) on four packed cells at once: the byte values
// are rebased so that live stamps map to [0, K') and tested in 16-bit slots
// (see LiveCfg); the rebasing constants are computed per slot from the clock.
//
// Windows longer than 254 slots (the paper's k up to 65534, Sec. 3.2) take
// 16-bit cells: stamp 1 + (s mod 65535), the same rules modulo 65535.
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <atomic>
#include <initializer_list>
#include <utility>

#include "internal.h"

namespace ssd {

// ---------------------------------------------------------------- helpers

__device__ __forceinline__ uint32_t tab_hash(const uint32_t* t, uint32_t x)
{
    // simple tabulation hashing: four byte-indexed tables XORed (Sec. 3.2, 3.3)
    return t[x & 255u] ^ t[256u + ((x >> 8) & 255u)] ^ t[512u + ((x >> 16) & 255u)] ^ t[768u + (x >> 24)];
}

__device__ __forceinline__ uint32_t shr32(uint32_t x, uint32_t s) { return s < 32u ? (x >> s) : 0u; }

__device__ __forceinline__ uint32_t wave_sum(uint32_t v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Reserve `cnt` consecutive slots of a device-wide list for this thread of a
// 256-thread block (every thread must call it): one atomic per block.
__device__ __forceinline__ unsigned long long block_append_256(uint32_t cnt, unsigned long long* counter)
{
    __shared__ uint32_t wtot[4];
    __shared__ unsigned long long bbase;
    const uint32_t lane = threadIdx.x & 63u, wid = threadIdx.x >> 6;
    uint32_t incl = cnt;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        uint32_t v = __shfl_up(incl, o, 64);
        if (lane >= (uint32_t)o) incl += v;
    }
    if (lane == 63) wtot[wid] = incl;
    __syncthreads();
    if (threadIdx.x == 0) {
        const uint32_t tot = wtot[0] + wtot[1] + wtot[2] + wtot[3];
        bbase = tot ? atomicAdd(counter, (unsigned long long)tot) : 0ull;
    }
    __syncthreads();
    uint32_t woff = 0;
    for (uint32_t w = 0; w < wid; w++) woff += wtot[w];
    const unsigned long long base = bbase;
    __syncthreads();
    return base + woff + (incl - cnt);
}

// Live cells of a 32-bit word of four cells: bits 8, 24 (bytes 0, 2) and
// 9, 25 (bytes 1, 3) are set for live cells.
__device__ __forceinline__ uint32_t live_bits(uint32_t w, const LiveCfg& L)
{
    const uint32_t M = 0x00FF00FFu, H = 0x01000100u;
    const uint32_t e = w & M, o = (w >> 8) & M;
    const uint32_t be = ((e + L.c1) & M) + L.c2;   // bit 8 of a slot: rebased stamp >= K'
    const uint32_t bo = ((o + L.c1) & M) + L.c2;
    uint32_t live = (~be & H) | ((~bo & H) << 1);
    if (L.wrap) live &= ((e + M) & H) | (((o + M) & H) << 1);   // exclude empty cells
    return live;
}

// The live cells of a 16-byte chunk as a 16-bit mask (bit i = cell i).
__device__ __forceinline__ uint32_t live_mask16(const uint4& v, const LiveCfg& L)
{
    auto nib = [](uint32_t x) { return ((x >> 8) & 3u) | ((x >> 22) & 12u); };
    return nib(live_bits(v.x, L)) | (nib(live_bits(v.y, L)) << 4) | (nib(live_bits(v.z, L)) << 8) |
           (nib(live_bits(v.w, L)) << 12);
}

// The word with every dead non-empty cell cleared (distance >= k).
__device__ __forceinline__ uint32_t expire_word(uint32_t w, const LiveCfg& L)
{
    const uint32_t M = 0x00FF00FFu;
    const uint32_t e = w & M, o = (w >> 8) & M;
    const uint32_t be = ((e + L.c1) & M) + L.c2;
    const uint32_t bo = ((o + L.c1) & M) + L.c2;
    const uint32_t de = ((be >> 8) & 0x00010001u) * 0xFFu;
    const uint32_t dd = (((bo >> 8) & 0x00010001u) * 0xFFu) << 8;
    return w & ~(de | dd);
}

// 16-bit cells: c is live iff (c - lo) mod 2^16 < K' and, when the live
// stamps wrap past 65535, c is not empty (LiveCfg c1 = lo, c2 = K').
__device__ __forceinline__ uint32_t live_cell16(uint32_t c, const LiveCfg& L)
{
    return (((c - L.c1) & 0xFFFFu) < L.c2 && (!L.wrap || c != 0u)) ? 1u : 0u;
}

// The live cells of a 16-byte chunk of eight 16-bit cells (bit i = cell i).
__device__ __forceinline__ uint32_t live_mask8_c16(const uint4& v, const LiveCfg& L)
{
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
    uint32_t m = 0;
#pragma unroll
    for (int i = 0; i < 4; i++)
        m |= (live_cell16(w[i] & 0xFFFFu, L) << (2 * i)) | (live_cell16(w[i] >> 16, L) << (2 * i + 1));
    return m;
}

// Two 16-bit cells with every dead non-empty one cleared (distance >= k).
__device__ __forceinline__ uint32_t expire_word16(uint32_t w, const LiveCfg& L)
{
    const uint32_t lo = w & 0xFFFFu, hi = w >> 16;
    return (live_cell16(lo, L) ? lo : 0u) | ((live_cell16(hi, L) ? hi : 0u) << 16);
}

// Index of the link owning flattened item g: the largest l with prefix[l] <= g
// (empty links have prefix[l] == prefix[l+1] and are skipped).
template <class U>
__device__ __forceinline__ uint32_t find_link(const U* prefix, uint32_t n_links, uint64_t g)
{
    uint32_t lo = 0, hi = n_links;
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (prefix[mid] <= g) lo = mid;
        else hi = mid;
    }
    return lo;
}

// A 16-byte load of memory that is streamed once (non-temporal: it takes no
// place in the caches from what is used again).
__device__ __forceinline__ uint4 load_stream(const uint4* p)
{
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
    return make_uint4(v.x, v.y, v.z, v.w);
}

__device__ __forceinline__ uint32_t uniform(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }

__device__ __forceinline__ void block_exclusive_scan_u64_1024(unsigned long long v, unsigned long long* lds /*[1024]*/,
                                                              unsigned long long* excl, unsigned long long* total)
{
    lds[threadIdx.x] = v;
    __syncthreads();
    for (uint32_t o = 1; o < 1024u; o <<= 1) {
        const unsigned long long t = threadIdx.x >= o ? lds[threadIdx.x - o] : 0ull;
        __syncthreads();
        lds[threadIdx.x] += t;
        __syncthreads();
    }
    *excl = lds[threadIdx.x] - v;
    *total = lds[1023];
    __syncthreads();
}

// Workgroup barrier that orders LDS only: global stores issued before it stay
// in flight (a plain __syncthreads waits for their completion).
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// LOCAL: only LDS is ordered by its barriers.
template <bool LOCAL = false>
__device__ __forceinline__ uint32_t block_exclusive_scan_1024(uint32_t v, uint32_t* lds /*[16]*/, uint32_t* total)
{
    const uint32_t lane = threadIdx.x & 63u, wid = threadIdx.x >> 6;
    uint32_t incl = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        uint32_t t = __shfl_up(incl, o, 64);
        if (lane >= (uint32_t)o) incl += t;
    }
    if (lane == 63) lds[wid] = incl;
    if (LOCAL) lds_barrier();
    else __syncthreads();
    uint32_t off = 0, tot = 0;
    for (uint32_t w = 0; w < 16; w++) {
        uint32_t x = lds[w];
        off += w < wid ? x : 0u;
        tot += x;
    }
    if (LOCAL) lds_barrier();
    else __syncthreads();
    *total = tot;
    return off + incl - v;
}

// ---------------------------------------------------------------- fill / clock

__global__ void k_fill_u32(uint32_t* p, uint64_t n, uint32_t v)
{
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = v;
}

// Per-slice constants of every link from its slot clock (grid: links x 16,
// thread 0 of block (l, 0)), and the hot bitmasks cleared for this close.
__global__ __launch_bounds__(256) void k_prepare(LinkDesc* links)
{
    const uint32_t l = blockIdx.x;
    const LinkDesc* D = links + l;
    uint32_t* p = reinterpret_cast<uint32_t*>(D->hotbits);     // hotT follows hotbits
    const uint64_t n = D->hot_words;
    for (uint64_t i = blockIdx.y * 256u + threadIdx.x; i < n; i += 256u * gridDim.y) p[i] = 0u;
    if (blockIdx.y != 0 || threadIdx.x != 0) return;
    const unsigned long long t = links[l].clock->t;
    const uint32_t k = links[l].k;
    const bool cell16 = links[l].cell16 != 0u;
    const uint32_t cur = slot_stamp(t, cell16);
    links[l].cur = cur;
    links[l].L = live_cfg(cur, k, cell16);
    const uint32_t period = expire_period(k, cell16);
    links[l].expire_period = period;
    links[l].expire_phase = (uint32_t)(t % period);
}

// A slot that only advances (one detector): the dead cells of this slot's
// expiry phase cleared, a wave per estimator, and the clock moved.  The slot's
// constants come with the launch, so that it is the only one (a launch for
// them, one for the expiry and one for the clock were 8.8 us and three
// launches for 320 MiB).
template <bool C16>
__global__ __launch_bounds__(256) void k_expire(ExpireArgs a)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) a.clock->t += 1ull;
    const uint32_t lane = threadIdx.x & 63u;
    const uint64_t s = a.phase + ((uint64_t)blockIdx.x * 4u + (threadIdx.x >> 6)) * a.period;
    if (s >= a.n_se) return;
    const uint32_t chunks = a.chunks;                // of 16 bytes, at least 64
    uint4* se = reinterpret_cast<uint4*>(a.state) + s * chunks;
    for (uint32_t c0 = lane; c0 < chunks; c0 += 256u) {
        uint4 v[4];
#pragma unroll
        for (uint32_t u = 0; u < 4; u++) v[u] = se[c0 + 64u * u < chunks ? c0 + 64u * u : c0];
#pragma unroll
        for (uint32_t u = 0; u < 4; u++) {
            if (c0 + 64u * u >= chunks) continue;
            uint4 n;
            n.x = C16 ? expire_word16(v[u].x, a.L) : expire_word(v[u].x, a.L);
            n.y = C16 ? expire_word16(v[u].y, a.L) : expire_word(v[u].y, a.L);
            n.z = C16 ? expire_word16(v[u].z, a.L) : expire_word(v[u].z, a.L);
            n.w = C16 ? expire_word16(v[u].w, a.L) : expire_word(v[u].w, a.L);
            if (n.x != v[u].x || n.y != v[u].y || n.z != v[u].z || n.w != v[u].w) se[c0 + 64u * u] = n;
        }
    }
}

// Copy every link's control block into one contiguous array (links whose
// blocks live in separate allocations).
__global__ void k_gather_ctl(const LinkDesc* links, uint32_t n_links, Ctl* dst)
{
    const uint32_t l = blockIdx.x * blockDim.x + threadIdx.x;
    if (l < n_links) dst[l] = *links[l].ctl;
}

// ---------------------------------------------------------------- scan
// Alg. 2 for every pair: one byte store per row.  `se_lo..se_hi` restricts
// the stores to one estimator window so that a pass's random stores stay in
// the last-level cache.

template <class T>
__device__ __forceinline__ void scan_pair(const uint32_t* tab, uint2 pr, T* state, uint32_t q, uint32_t delta,
                                          uint32_t log2eta, uint32_t row_lo, uint32_t row_hi, uint64_t se_lo,
                                          uint64_t se_hi, T stamp)
{
    const uint32_t qmask = (1u << q) - 1u;
    const uint32_t d = tab_hash(tab + 1024, pr.y) & ((1u << log2eta) - 1u);   // H1(oip)
    const uint32_t h0 = tab_hash(tab, pr.x) & qmask;                          // RHFG[0](cip)
    for (uint32_t i = row_lo; i < row_hi; i++) {
        const uint32_t col = i == 0 ? h0 : ((shr32(pr.x, (i - 1) * delta) ^ h0) & qmask);
        const uint64_t se = ((uint64_t)i << q) | col;
        if (se >= se_lo && se < se_hi) state[(se << log2eta) | d] = stamp;
    }
}

// Whether a call of r rows is scanned by eighths, from 64 of its hosts, one a
// lane, the same for every workgroup: not where few hosts bring much of the
// call (a quarter, half from eight rows on), whose stores fall into few lines
// that a shared window also keeps in the L2s.  Up to eight hosts of three
// lanes or more are looked for.  Six rows, a million pairs into 24 MiB, shared
// and by eighths: of as many hosts 77 and 72 us, Pareto 73 and 45, a fifth of
// one host 61 and 61, half 42 and 46, ten hosts 28 and 53, one 16 and 38.
// Eight rows, half of one host, 16 MiB: 54 and 49.
__device__ __forceinline__ bool by_eighths(uint32_t host, uint32_t r)
{
    uint64_t left = ~0ull;
    uint32_t heavy = 0;
    for (uint32_t g = 0; g < 8u && left; g++) {
        const uint64_t same = __ballot(host == (uint32_t)__builtin_amdgcn_readlane((int)host, __ffsll((long long)left) - 1)) & left;
        const uint32_t c = (uint32_t)__popcll(same);
        if (c > 2u) heavy += c;
        left &= ~same;
    }
    return heavy <= (r < 8u ? 16u : 32u);
}

// By eighths (a.eighths, and the call's hosts: by_eighths) workgroup g stores
// only into eighth g mod 8 of the pass's window.  Workgroup g runs on XCD g mod
// 8, so every XCD stores into a range that its own L2 holds, where a window that all eight share is stored into
// the Infinity Cache at 83 G/s (each L2 writes back its own bytes of a line).
// Every XCD reads and hashes all pairs for it, which now bounds it (eight LDS
// table lookups a pair), but takes only the one or two rows of its eighth.
// (Results do not depend on the placement.)
template <class T>
__global__ __launch_bounds__(256) void k_scan(ScanArgs a)
{
    __shared__ uint32_t tab[2048];
    const uint32_t sample = a.eighths ? a.pairs[(threadIdx.x & 63u) * (a.n >> 6)].x : 0u;
    for (uint32_t i = threadIdx.x; i < 2048u; i += 256u) tab[i] = a.tables[i];
    __syncthreads();
    uint64_t se_lo = a.se_lo, se_hi = a.se_hi;
    uint32_t g = blockIdx.x, grid = gridDim.x;
    if (a.eighths && by_eighths(sample, (uint32_t)(a.se_hi >> a.q))) {
        const uint64_t per = (a.se_hi - a.se_lo + 7u) >> 3;
        se_lo = min(a.se_hi, a.se_lo + (g & 7u) * per);
        se_hi = min(a.se_hi, se_lo + per);
        if (se_lo == se_hi) return;
        g >>= 3;
        grid >>= 3;
    }
    const uint32_t row_lo = (uint32_t)(se_lo >> a.q);
    const uint32_t row_hi = (uint32_t)((se_hi - 1) >> a.q) + 1u;
    const uint64_t stride = (uint64_t)grid * 256u;
    for (uint64_t p = (uint64_t)g * 256u + threadIdx.x; p < a.n; p += stride)
        scan_pair<T>(tab, a.pairs[p], reinterpret_cast<T*>(a.state), a.q, a.delta, a.log2eta, row_lo, row_hi,
                     se_lo, se_hi, (T)a.stamp);
}

// Adds v to counter i (v depends on i alone) for the lanes that `on` holds
// for.  A heavy host's pairs move the same counters, and atomics of one
// address pass one after another: one lane adds for all of a wave that move
// the same counter, counter by counter, up to 12 of them and until two were
// moved by a lane alone (light hosts, whose lanes then add for themselves).
// 65535 pairs of one host into each of 8 links of 384 MiB, eta = 16384: 852 us
// with an atomic a lane, 435 so; of ten hosts 646 and 478; of as many hosts as
// pairs 413 and 423.
constexpr uint32_t COUNT_GROUPS = 12, COUNT_ALONE = 2;
__device__ __forceinline__ void add_counts(uint32_t* counts, uint32_t i, uint32_t v, bool on)
{
    const uint32_t lane = threadIdx.x & 63u;
    uint64_t left = __ballot(on);
    for (uint32_t g = 0, alone = 0; g < COUNT_GROUPS && alone < COUNT_ALONE && left; g++) {
        const uint32_t first = (uint32_t)__ffsll((long long)left) - 1u;
        const uint64_t same = __ballot(on && i == (uint32_t)__builtin_amdgcn_readlane((int)i, (int)first)) & left;
        if (lane == first) atomicAdd(&counts[i], v * (uint32_t)__popcll(same));
        left &= ~same;
        if (!(same & (same - 1ull))) alone++;
    }
    if ((left >> lane) & 1ull) atomicAdd(&counts[i], v);
}

// The same keeping exact counters exact, for calls with so few offsets that a
// workgroup per bin costs more than they do: every cell's stamp is exchanged
// by a compare-and-swap of its 32-bit word, and the one thread that changes it
// moves its estimator's counters in memory (which slot, see k_apply_counted).
// Six rows in flight.  Bound by random device-wide atomics, three for a cell
// not yet stamped in the slice (the exchange, and a counter up and one down or
// the total up; more exchanges where threads meet in a word), 19 to 27 G/s:
// 5.8 G offsets/s.
__device__ __forceinline__ void scan_pair_counted(const uint32_t* tab, uint2 pr, const LinkDesc* D, uint32_t stamp,
                                                  uint32_t slot)
{
    const uint32_t q = D->q, delta = D->delta, log2eta = D->log2eta, r = D->r, k = D->k;
    const uint32_t qmask = (1u << q) - 1u, n_se = (uint32_t)D->n_se;
    uint32_t* words = reinterpret_cast<uint32_t*>(D->state);
    const uint32_t d = tab_hash(tab + 1024, pr.y) & ((1u << log2eta) - 1u);   // H1(oip)
    const uint32_t h0 = tab_hash(tab, pr.x) & qmask;                          // RHFG[0](cip)
    const uint32_t sh = (d & 3u) * 8u;
    for (uint32_t i0 = 0; i0 < r; i0 += 6u) {
        uint64_t se[6];
        uint32_t w[6];
#pragma unroll
        for (uint32_t u = 0; u < 6; u++) {
            const uint32_t i = min(i0 + u, r - 1u);
            const uint32_t col = i == 0 ? h0 : ((shr32(pr.x, (i - 1) * delta) ^ h0) & qmask);
            se[u] = ((uint64_t)i << q) | col;
            w[u] = __hip_atomic_load(words + (((se[u] << log2eta) | d) >> 2), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        uint32_t left = (1u << min(6u, r - i0)) - 1u;          // rows not yet stamped
        while (left) {
            uint32_t was[6];
#pragma unroll
            for (uint32_t u = 0; u < 6; u++) {
                was[u] = w[u];
                if (!((left >> u) & 1u)) continue;
                if (((w[u] >> sh) & 0xFFu) == stamp) left &= ~(1u << u);
                else was[u] = atomicCAS(words + (((se[u] << log2eta) | d) >> 2), w[u], (w[u] & ~(0xFFu << sh)) | (stamp << sh));
            }
#pragma unroll
            for (uint32_t u = 0; u < 6; u++) {
                if (!((left >> u) & 1u)) continue;
                const bool mine = was[u] == w[u];              // this thread's stamp
                const uint32_t b = (w[u] >> sh) & 0xFFu, age = (stamp + 255u - b) % 255u;
                const bool live = b && age < k;
                const uint32_t at = live ? (slot >= age ? slot - age : slot + k - age) : k;
                add_counts(D->counts, slot * n_se + (uint32_t)se[u], 1u, mine);
                add_counts(D->counts, at * n_se + (uint32_t)se[u], live ? ~0u : 1u, mine);
                if (mine) left &= ~(1u << u);
                w[u] = was[u];
            }
        }
    }
}

__global__ __launch_bounds__(256) void k_scan_counted(const LinkDesc* D, const uint2* pairs, uint64_t n, uint32_t stamp,
                                                      uint32_t slot)
{
    __shared__ uint32_t tab[2048];
    for (uint32_t i = threadIdx.x; i < 2048u; i += 256u) tab[i] = D->tables[i];
    __syncthreads();
    const uint64_t stride = (uint64_t)gridDim.x * 256u;
    for (uint64_t p = (uint64_t)blockIdx.x * 256u + threadIdx.x; p < n; p += stride) scan_pair_counted(tab, pairs[p], D, stamp, slot);
}

// Persistent scan over many links: workgroups pull tile numbers from a device
// counter; a tile is some pairs of one link restricted to one estimator
// window, found by binary search over the windows' tile prefix.  Windows are
// ordered by state address and tiles are small, so the tiles in flight store
// into a cache-sized range of state; a workgroup reloads the tabulation
// tables only when its link changes.  Every workgroup leaves once the counter
// passes the last tile.
__global__ __launch_bounds__(256) void k_scan_tiles(TileScanArgs a)
{
    __shared__ uint32_t tab[2048];
    __shared__ unsigned long long next;
    uint32_t loaded = 0xFFFFFFFFu;
    for (;;) {
        if (threadIdx.x == 0) next = atomicAdd(a.counter, 1ull);
        __syncthreads();
        const unsigned long long t = next;
        __syncthreads();
        if (t >= a.n_tiles) break;
        uint32_t lo = 0, hi = a.n_wins;
        while (hi - lo > 1) {
            const uint32_t mid = (lo + hi) >> 1;
            if (a.wins[mid].tile_base <= t) lo = mid;
            else hi = mid;
        }
        const ScanWindow W = a.wins[lo];
        const uint64_t first = W.start + (t - W.tile_base) * W.tile;
        const uint64_t last = min(first + W.tile, W.start + W.n);
        const LinkDesc* D = a.links + W.link;
        if (W.link != loaded) {
            for (uint32_t i = threadIdx.x; i < 2048u; i += 256u) tab[i] = D->tables[i];
            __syncthreads();
            loaded = W.link;
        }
        if (W.counted) {
            for (uint64_t p = first + threadIdx.x; p < last; p += 256u) scan_pair_counted(tab, a.pairs[p], D, W.stamp, W.slot);
            continue;
        }
        const uint32_t q = D->q, delta = D->delta, log2eta = D->log2eta;
        uint8_t* state = D->state;
        const uint32_t row_lo = (uint32_t)(W.se_lo >> q);
        const uint32_t row_hi = (uint32_t)((W.se_hi - 1) >> q) + 1u;
        for (uint64_t p = first + threadIdx.x; p < last; p += 256u)
            scan_pair<uint8_t>(tab, a.pairs[p], state, q, delta, log2eta, row_lo, row_hi, W.se_lo, W.se_hi,
                               (uint8_t)W.stamp);
    }
}

// ---------------------------------------------------------------- binned scan
// Alg. 2 in two steps, for states much larger than the caches.
// k_bin: each workgroup takes `pb` pairs, computes their r cell addresses and
// counting-sorts the bin-local offsets by state bin (bins of 2^bin_shift
// bytes) in LDS, then writes them as one coalesced segment; the start of every
// bin in the segment goes to a bin-major table.
// k_apply: the byte stores, bin by bin.  Workgroup g runs on XCD g mod 8 (the
// dispatcher deals workgroups to the XCDs in turn) and the bins of an XCD are
// visited in ascending order by all its workgroups together, so the stores of
// each XCD land in a range its own L2 holds.  Results do not depend on the
// placement: every store is independent.

__device__ __forceinline__ void pair_hashes(const uint32_t* tab, uint2 pr, uint32_t q, uint32_t log2eta,
                                            uint32_t* h0, uint32_t* d)
{
    *d = tab_hash(tab + 1024, pr.y) & ((1u << log2eta) - 1u);   // H1(oip)
    *h0 = tab_hash(tab, pr.x) & ((1u << q) - 1u);               // RHFG[0](cip)
}

// Row i's estimator of a pair.  A bin holds whole estimators (2^(bin_shift -
// log2eta) of them), so the bin and the offset in it come from the estimator's
// number in 32 bits (64-bit cell addresses cost k_bin 2 %).
__device__ __forceinline__ uint32_t estimator(uint32_t x, uint32_t i, uint32_t h0, uint32_t q, uint32_t delta)
{
    const uint32_t col = i == 0 ? h0 : ((shr32(x, (i - 1) * delta) ^ h0) & ((1u << q) - 1u));
    return (i << q) | col;
}

// The segments (chunks of pairs) of a binning workgroup: workgroup g runs on
// XCD g mod 8, which takes a contiguous eighth of the segments, so that the
// bin table entries of neighbouring segments, which share sectors, are
// written through one L2 and leave it merged; the XCD's workgroups take its
// segments in turn, a.rounds each at most.
struct BinSegments {
    uint32_t at, end, step;
};
__device__ __forceinline__ BinSegments bin_segments(const BinArgs& a, uint32_t g)
{
    const uint32_t per = (a.blocks + 7u) >> 3, first = (g & 7u) * per;
    return {first + (g >> 3), min(first + per, a.blocks), (per + a.rounds - 1u) / a.rounds};
}

// A workgroup's sorted offsets out to its segment, coalesced: 4 bytes each, or
// (bins of at most 2 MiB) three 21-bit offsets per 8-byte word.
__device__ __forceinline__ void write_segment(const BinArgs& a, uint32_t sg, const uint32_t* stage, uint32_t n)
{
    const uint64_t seg_items = (uint64_t)a.pb * a.r;
    if (a.pack) {
        uint64_t* seg = reinterpret_cast<uint64_t*>(a.items) + (uint64_t)sg * packed_seg_words(seg_items);
        for (uint32_t w = threadIdx.x; w * 3u < n; w += 1024u) {
            const uint32_t i = w * 3u;
            uint64_t v = stage[i];
            if (i + 1 < n) v |= (uint64_t)stage[i + 1] << 21;
            if (i + 2 < n) v |= (uint64_t)stage[i + 2] << 42;
            seg[w] = v;
        }
    } else {
        uint32_t* seg = a.items + (uint64_t)sg * seg_items;
        for (uint32_t i = threadIdx.x; i < n; i += 1024u) seg[i] = stage[i];
    }
}

// Item i of segment j as written by write_segment.
__device__ __forceinline__ uint32_t read_item(const ApplyArgs& a, uint32_t j, uint32_t i)
{
    if (a.pack) {
        const uint64_t w = reinterpret_cast<const uint64_t*>(a.items)[(uint64_t)j * packed_seg_words(a.seg) + i / 3u];
        return (uint32_t)(w >> (21u * (i % 3u))) & 0x1FFFFFu;
    }
    return a.items[(uint64_t)j * a.seg + i];
}

// Up to 160 KiB of LDS per workgroup: about 6000 pairs, so that the run of
// one bin in one segment is long (about 50 offsets at 2 MiB bins) and
// k_apply's reads of the runs are dense.  Pass 1 counts the bins' offsets,
// pass 2 hashes again and places each offset at its bin's next free slot.
// (workgroup g of this link's launch; lds: the dynamic LDS, wsum: 16 words)
__device__ __forceinline__ void bin_generic(const BinArgs& a, uint32_t sg, uint32_t* lds, uint32_t* wsum)
{
    uint32_t* tab = lds;
    uint32_t* hist = lds + 2048;
    uint32_t* stage = hist + a.n_bins + 1;
    for (uint32_t i = threadIdx.x; i < 2048u; i += 1024u) tab[i] = a.tables[i];
    for (uint32_t i = threadIdx.x; i <= a.n_bins; i += 1024u) hist[i] = 0u;
    __syncthreads();
    const uint64_t p0 = (uint64_t)sg * a.pb;
    const uint32_t np = (uint32_t)min((uint64_t)a.pb, a.n - p0);
    const uint32_t q = a.q, r = a.r, delta = a.delta, log2eta = a.log2eta, es = a.bin_shift - log2eta;
    const uint32_t emask = (1u << es) - 1u;
    for (uint32_t p = threadIdx.x; p < np; p += 1024u) {
        const uint2 pr = a.pairs[p0 + p];
        uint32_t h0, d;
        pair_hashes(tab, pr, q, log2eta, &h0, &d);
        for (uint32_t i = 0; i < r; i++) atomicAdd(&hist[estimator(pr.x, i, h0, q, delta) >> es], 1u);
    }
    __syncthreads();
    const uint32_t per = (a.n_bins + 1023u) / 1024u;
    const uint32_t b0 = min(a.n_bins, threadIdx.x * per), b1 = min(a.n_bins, b0 + per);
    uint32_t sum = 0;
    for (uint32_t b = b0; b < b1; b++) sum += hist[b];
    uint32_t total;
    uint32_t start = block_exclusive_scan_1024(sum, wsum, &total);
    for (uint32_t b = b0; b < b1; b++) {
        const uint32_t c = hist[b];
        hist[b] = start;
        a.table[(uint64_t)b * a.blocks + sg] = start;
        start += c;
    }
    if (threadIdx.x == 0) a.table[(uint64_t)a.n_bins * a.blocks + sg] = np * r;
    __syncthreads();
    for (uint32_t p = threadIdx.x; p < np; p += 1024u) {
        const uint2 pr = a.pairs[p0 + p];
        uint32_t h0, d;
        pair_hashes(tab, pr, q, log2eta, &h0, &d);
        for (uint32_t i = 0; i < r; i++) {
            const uint32_t se = estimator(pr.x, i, h0, q, delta);
            stage[atomicAdd(&hist[se >> es], 1u)] = ((se & emask) << log2eta) | d;
        }
    }
    __syncthreads();
    write_segment(a, sg, stage, np * r);
}

// Segment sg's pairs, PPT per thread (past the end: the last pair).
template <int PPT>
__device__ __forceinline__ void load_pairs(const BinArgs& a, uint32_t sg, uint2* pr)
{
    const uint64_t p0 = (uint64_t)sg * a.pb;
    const uint32_t np = (uint32_t)min((uint64_t)a.pb, a.n - p0);
#pragma unroll
    for (int u = 0; u < PPT; u++) pr[u] = a.pairs[p0 + min(threadIdx.x + u * 1024u, np - 1u)];
}

// The same sort for the common row counts (R rows, up to PPT pairs per thread)
// with the hashes of every pair and each offset's rank in its bin (of the
// count pass) kept in registers between the two passes; bins and offsets are
// cheap to form again, and kept instead they left no registers to load ahead.
// PIPE: a workgroup sorts its segments one after another, and the pairs of
// the next are loaded while this one is placed and written; no barrier waits
// for them or for the segment's stores.  (6 M pairs of six rows: 97 us with a
// workgroup per segment, 69 so: the loads were 29 of them.  The phases now
// follow one another in every compute unit: hashing, the counts in LDS, the
// scan with the table's stores, the placing and the writing take about a
// fifth each.  Workgroups of half a compute unit overlap each other's loads
// and take one segment: 2.7 M pairs of five rows 26.5 us, in turn 28.)
template <int R, int PPT, bool PIPE>
__device__ __forceinline__ void bin_reg(const BinArgs& a, uint32_t g, uint32_t* lds, uint32_t* wsum)
{
    const BinSegments S = bin_segments(a, g);
    if (S.at >= S.end) return;
    uint32_t* tab = lds;
    uint32_t* hist = lds + 2048;
    uint32_t* stage = hist + a.n_bins + 1;
    uint2 pr[PPT];
    load_pairs<PPT>(a, S.at, pr);
    for (uint32_t i = threadIdx.x; i < 2048u; i += 1024u) tab[i] = a.tables[i];
    const uint32_t q = a.q, delta = a.delta, log2eta = a.log2eta, es = a.bin_shift - log2eta;
    const uint32_t emask = (1u << es) - 1u;
    const uint32_t per = (a.n_bins + 1023u) / 1024u;
    const uint32_t b0 = min(a.n_bins, threadIdx.x * per), b1 = min(a.n_bins, b0 + per);
    for (uint32_t sg = S.at; sg < S.end; sg += S.step) {
        const uint32_t np = (uint32_t)min((uint64_t)a.pb, a.n - (uint64_t)sg * a.pb);
        for (uint32_t i = threadIdx.x; i <= a.n_bins; i += 1024u) hist[i] = 0u;
        lds_barrier();               // (also: the segment before has left the staging)
        uint32_t x[PPT], h0[PPT], d[PPT], rank[PPT][(R + 1) / 2];
#pragma unroll
        for (int u = 0; u < PPT; u++) {
            if (threadIdx.x + u * 1024u >= np) continue;
            x[u] = pr[u].x;
            pair_hashes(tab, pr[u], q, log2eta, &h0[u], &d[u]);
#pragma unroll
            for (int i = 0; i < R; i++) {
                const uint32_t at = atomicAdd(&hist[estimator(x[u], i, h0[u], q, delta) >> es], 1u);
                if (i & 1) rank[u][i / 2] |= at << 16;
                else rank[u][i / 2] = at;
            }
        }
        if (PIPE && sg + S.step < S.end) load_pairs<PPT>(a, sg + S.step, pr);
        lds_barrier();
        uint32_t sum = 0;
        for (uint32_t b = b0; b < b1; b++) sum += hist[b];
        uint32_t total;
        uint32_t start = block_exclusive_scan_1024<true>(sum, wsum, &total);
        for (uint32_t b = b0; b < b1; b++) {
            const uint32_t c = hist[b];
            hist[b] = start;
            a.table[(uint64_t)b * a.blocks + sg] = start;
            start += c;
        }
        if (threadIdx.x == 0) a.table[(uint64_t)a.n_bins * a.blocks + sg] = np * R;
        lds_barrier();
#pragma unroll
        for (int u = 0; u < PPT; u++) {
            if (threadIdx.x + u * 1024u >= np) continue;
#pragma unroll
            for (int i = 0; i < R; i++) {
                const uint32_t se = estimator(x[u], i, h0[u], q, delta);
                const uint32_t at = (i & 1) ? rank[u][i / 2] >> 16 : rank[u][i / 2] & 0xFFFFu;
                stage[hist[se >> es] + at] = ((se & emask) << log2eta) | d[u];
            }
        }
        lds_barrier();
        write_segment(a, sg, stage, np * R);
        if (!PIPE) return;
    }
}

// The general binning of a workgroup's segments.
__device__ __forceinline__ void bin_any(const BinArgs& a, uint32_t g, uint32_t* lds, uint32_t* wsum)
{
    const BinSegments S = bin_segments(a, g);
    for (uint32_t sg = S.at; sg < S.end; sg += S.step) {
        bin_generic(a, sg, lds, wsum);
        __syncthreads();
    }
}

// R = 0: the general binning; else the register binning of R rows.  HALF: the
// workgroup's LDS and registers are at most half a compute unit's, so that two
// share it and one's loads and barriers overlap the other's LDS work: LDS
// is active less than half of a full-size workgroup's time.  64 links' 23 M
// pairs: 1246 us with whole segments, 1152 with halves where their runs are
// long enough (1020 with the register sort as it is now); 6 M pairs of five
// rows into 320 MiB of 16-bit cells 64 and 55 (52).
template <int R, int PPT, bool HALF>
__global__ __launch_bounds__(1024, HALF ? 8 : 4) void k_bin(BinArgs a)
{
    extern __shared__ uint32_t lds[];
    __shared__ uint32_t wsum[16];
    if constexpr (R == 0) bin_any(a, blockIdx.x, lds, wsum);
    else bin_reg<R, PPT, !HALF>(a, blockIdx.x, lds, wsum);
}

// Several links in one launch: workgroup g belongs to the link whose range
// of the workgroup prefix holds it.  Every link's range is a multiple of 8
// workgroups, so that the dealing of its segments to XCDs is the one of a
// launch of its own.  Each workgroup takes its link's binning variant (the
// register binning of five or six rows where the segment fits it, else the
// general one); the launch keeps the larger register count of the two.  The
// links whose segments leave room for two workgroups on a compute unit (HALF)
// take a launch of their own.
template <bool HALF>
__global__ __launch_bounds__(1024, HALF ? 8 : 4) void k_bin_multi_rows(MultiBinArgs m)
{
    extern __shared__ uint32_t lds[];
    __shared__ uint32_t wsum[16];
    const uint32_t l = uniform(find_link(m.wg_prefix, m.n, blockIdx.x));
    const BinArgs a = m.args[l];
    const uint32_t g = blockIdx.x - m.wg_prefix[l];
    constexpr int P6 = HALF ? 3 : 6, P5 = HALF ? 4 : 7;
    if (a.r == 6 && a.pb <= P6 * 1024u) bin_reg<6, P6, !HALF>(a, g, lds, wsum);
    else if (a.r == 5 && a.pb <= P5 * 1024u) bin_reg<5, P5, !HALF>(a, g, lds, wsum);
    else bin_any(a, g, lds, wsum);
}

// One wave per workgroup.  Workgroup g: XCD g mod 8, the (g mod 8) + 8 * (w /
// parts)-th bin from the top with w = g / 8, segments [part * per_part, ...),
// 64 segments per round: lane j holds segment j's run of the bin, and the
// wave walks the concatenated runs 64 items at a time.
constexpr uint32_t APPLY_UNROLL = 2;      // items per lane in flight

template <bool PACK, class T>
__device__ __forceinline__ void apply_body(const ApplyArgs& a, uint32_t g)
{
    const uint64_t seg_words = PACK ? packed_seg_words(a.seg) : a.seg;   // item words per segment
    const uint32_t w = g >> 3;
    const uint32_t walk = (g & 7u) + 8u * (w / a.parts);
    if (walk >= a.n_bins) return;
    const uint32_t bin = a.n_bins - 1u - walk;     // highest bins first: the lowest stay cached for hot detection
    const uint32_t part = w % a.parts;
    const uint32_t lane = threadIdx.x;
    const uint32_t j0 = part * a.per_part;
    const uint32_t j1 = min(a.blocks, j0 + a.per_part);
    T* base = reinterpret_cast<T*>(a.state) + ((uint64_t)bin << a.bin_shift);    // bins count cells
    const T stamp = (T)a.stamp;
    const uint32_t* row = a.table + (uint64_t)bin * a.blocks;
    for (uint32_t jb = j0; jb < j1; jb += 64u) {
        const uint32_t j = jb + lane;
        uint32_t st = 0, c = 0;
        if (j < j1) {
            st = row[j];
            c = row[a.blocks + j] - st;
        }
        uint32_t incl = c;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t v = __shfl_up(incl, o, 64);
            if (lane >= (uint32_t)o) incl += v;
        }
        const uint32_t excl = incl - c;
        const uint32_t total = __shfl(incl, 63, 64);
        for (uint32_t t0 = 0; t0 < total; t0 += 64u * APPLY_UNROLL) {
            // every lane loads (past the end: the first word of segment jb),
            // so that the loads issue back to back and are waited for once
            uint32_t it[APPLY_UNROLL], sg[APPLY_UNROLL];
            bool ok[APPLY_UNROLL];
#pragma unroll
            for (int u = 0; u < (int)APPLY_UNROLL; u++) {
                const uint32_t t = t0 + (uint32_t)u * 64u + lane;
                // the run holding item t: the largest lane whose run starts at or before t
                uint32_t lo = 0;
#pragma unroll
                for (uint32_t sft = 32; sft > 0; sft >>= 1) {
                    const uint32_t e = __shfl(excl, (int)(lo + sft), 64);
                    if (e <= t) lo += sft;
                }
                const uint32_t rs = __shfl(st, (int)lo, 64);
                const uint32_t re = __shfl(excl, (int)lo, 64);
                ok[u] = t < total;
                it[u] = ok[u] ? rs + (t - re) : 0u;
                sg[u] = ok[u] ? jb + lo : jb;
            }
            uint64_t raw[APPLY_UNROLL];
#pragma unroll
            for (int u = 0; u < (int)APPLY_UNROLL; u++) {
                const uint64_t w = (uint64_t)sg[u] * seg_words + (PACK ? it[u] / 3u : it[u]);
                raw[u] = PACK ? reinterpret_cast<const uint64_t*>(a.items)[w] : (uint64_t)a.items[w];
            }
            // offsets taken on every lane and pinned before the first store (an
            // empty asm reading them), so that no load sinks into a store's
            // branch and waits for the stores before it
            uint32_t off[APPLY_UNROLL];
#pragma unroll
            for (int u = 0; u < (int)APPLY_UNROLL; u++) {
                off[u] = PACK ? (uint32_t)(raw[u] >> (21u * (it[u] % 3u))) & 0x1FFFFFu : (uint32_t)raw[u];
                asm volatile("" : : "v"(off[u]));
            }
#pragma unroll
            for (int u = 0; u < (int)APPLY_UNROLL; u++)
                if (ok[u]) base[off[u]] = stamp;
        }
    }
}

template <bool PACK, class T>
__global__ __launch_bounds__(64) void k_apply(ApplyArgs a)
{
    apply_body<PACK, T>(a, blockIdx.x);
}

// Several links in one launch (8-bit cells), as k_bin_multi.
template <bool PACK>
__global__ __launch_bounds__(64) void k_apply_multi(MultiApplyArgs m)
{
    const uint32_t l = uniform(find_link(m.wg_prefix, m.n, blockIdx.x));
    const ApplyArgs a = m.args[l];
    apply_body<PACK, uint8_t>(a, blockIdx.x - m.wg_prefix[l]);
}

// Counted variant: one workgroup per bin.  The walk over the bin's items only
// marks their cells in an LDS bitmap (a bit per cell); then every marked cell
// is visited once, 16-byte chunk by chunk: a cell whose stamp is not the open
// slice's yet takes it and moves in its estimator's per-slot counters (+1 for
// the open slot, -1 for the slot of an old stamp still in the window).
// Stamps of earlier launches into the same slice are recognised by their
// value, so every cell is counted once per slice.  The workgroup owns its
// bin's cells and estimators: chunks are written back whole, and the
// counters, summed in LDS, are added to memory by atomics whose result is
// unused (so that nothing waits for a read of the old values).
constexpr uint32_t CAPPLY_WAVES = 16;
constexpr uint32_t CAPPLY_CHUNKS = 4;     // bitmap words per thread in flight in the visit
constexpr uint32_t CAPPLY_LIST = 4096;    // marked words listed for the visit (more: the whole bitmap is swept)

// Add d to 16-bit counter i of the LDS counters (two biased halves per word;
// the halves never carry into each other, so a 32-bit add does it).
__device__ __forceinline__ void cnt_add(uint32_t* cw, uint32_t i, int d)
{
    atomicAdd(&cw[i >> 1], (uint32_t)d << ((i & 1u) * 16u));
}

// The marked cells of one 4-byte word (mask m, a bit per byte): the new
// stamps, the count of cells restamped, and -1 on the slot of every old stamp
// still in the window (counters ce0 + slot of the LDS counters cw).  Byte
// masks are formed SWAR; only the restamped cells with an old stamp are
// visited one by one.
__device__ __forceinline__ uint32_t stamp_word(uint32_t x, uint32_t m, uint32_t stamp, uint32_t k, uint32_t slot,
                                               uint32_t* cw, uint32_t ce0, uint32_t& changed)
{
    const uint32_t lanes = ((m * 0x00204081u) & 0x01010101u) * 0xFFu;       // bit i of m -> byte i
    const uint32_t y = x ^ (stamp * 0x01010101u);
    const uint32_t ne = ((((y & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | y) & 0x80808080u) >> 7;   // byte != stamp
    const uint32_t nz = ((((x & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | x) & 0x80808080u) >> 7;   // byte != 0
    const uint32_t chg = lanes & (ne * 0xFFu);
    changed += (uint32_t)__popc(chg) >> 3;
    uint32_t old = (chg & (nz * 0xFFu)) & 0x01010101u;      // restamped cells with an old stamp
    while (old) {
        const uint32_t i = ((uint32_t)__ffs(old) - 1u) >> 3;
        old &= old - 1u;
        const uint32_t b = (x >> (8u * i)) & 0xFFu;
        const uint32_t d = (stamp + 255u - b) % 255u;      // slices since the old stamp
        if (d < k) cnt_add(cw, ce0 + (slot >= d ? slot - d : slot + k - d), -1);
    }
    return (x & ~chg) | ((stamp * 0x01010101u) & chg);
}

// The first half of the bitmap stores (bin `bin` of this launch): the LDS is
// cleared -- its first bm_words words, the bitmap of the bin's cells, to 0,
// the rest of its n_words to 0x80008000 (two biased 16-bit counters) -- and
// every cell that an offset of the bin names is marked in the bitmap; a
// word's first mark appends it to list (the marked words, in the order they
// were first marked; n_list counts them all, also past CAPPLY_LIST).
__device__ __forceinline__ void mark_runs(const ApplyArgs& a, uint32_t bin, uint32_t* lds, uint32_t bm_words,
                                          uint32_t n_words, uint16_t* list, uint32_t& n_list)
{
    const uint32_t* row = a.table + (uint64_t)bin * a.blocks;
    // a run is shared by 2^ls lanes where there are fewer runs than threads
    // (64 links of 1 to 1024 runs a bin: 4275 us with a lane each, 4124 so)
    const uint32_t ls = a.blocks * 2u <= blockDim.x ? 31u - (uint32_t)__clz(blockDim.x / a.blocks) : 0u;
    const uint32_t part = threadIdx.x & ((1u << ls) - 1u);
    // this lane's first run (segment j), loaded before the LDS is cleared so
    // that the two overlap
    uint32_t j = threadIdx.x >> ls, st = 0, c = 0;
    if (j < a.blocks) {
        st = row[j];
        c = row[a.blocks + j] - st;
    }
    for (uint32_t i = threadIdx.x; i < n_words; i += blockDim.x) lds[i] = i < bm_words ? 0u : 0x80008000u;
    if (threadIdx.x == 0) n_list = 0u;
    __syncthreads();
    // walk: four aligned 16-byte loads (24 offsets) of the run at a time;
    // words past the segment's end are read from its last pair and fall
    // outside the run
    const uint64_t seg_words = packed_seg_words(a.seg);
    const uint64_t* items = reinterpret_cast<const uint64_t*>(a.items);
    const uint32_t last_pair = (uint32_t)(seg_words / 2u) - 1u;
    for (;;) {
        const uint32_t end = st + c;                                   // items [st, end)
        const uint32_t w_end = (end + 2u) / 3u;
        const uint4* seg = reinterpret_cast<const uint4*>(items + (uint64_t)min(j, a.blocks - 1u) * seg_words);
        for (uint32_t base = ((st / 3u) & ~1u) + 8u * part; c && base < w_end; base += 8u << ls) {
            uint4 q[4];
#pragma unroll
            for (int i = 0; i < 4; i++) q[i] = seg[min(base / 2u + (uint32_t)i, last_pair)];
#pragma unroll
            for (int i = 0; i < 8; i++) {
                const uint64_t wd = (i & 1) ? ((uint64_t)q[i / 2].w << 32 | q[i / 2].z)
                                            : ((uint64_t)q[i / 2].y << 32 | q[i / 2].x);
                const uint32_t i0 = 3u * (base + (uint32_t)i);
#pragma unroll
                for (uint32_t sft = 0; sft < 3; sft++) {
                    if (i0 + sft < st || i0 + sft >= end) continue;
                    const uint32_t off = (uint32_t)(wd >> (21u * sft)) & 0x1FFFFFu;
                    if (atomicOr(&lds[off >> 5], 1u << (off & 31u)) == 0u) {
                        const uint32_t at = atomicAdd(&n_list, 1u);
                        if (at < CAPPLY_LIST) list[at] = (uint16_t)(off >> 5);
                    }
                }
            }
        }
        j += blockDim.x >> ls;
        if (j >= a.blocks) break;
        st = row[j];
        c = row[a.blocks + j] - st;
    }
    __syncthreads();
}

// (workgroup g of this link's launch; lds: the dynamic LDS; list / n_list:
// the workgroup's list of marked words)
__device__ __forceinline__ void apply_counted_body(const ApplyArgs& a, uint32_t g, uint32_t* lds, uint16_t* list,
                                                   uint32_t& n_list, uint32_t* wsum)
{
    // workgroup g runs on XCD g mod 8, which takes a contiguous eighth of the
    // bins in order: neighbouring bins, whose runs share cache lines in every
    // segment, are read through the same L2 at about the same time
    const uint32_t per_xcd = (a.n_bins + 7u) >> 3;
    const uint32_t bin = (g & 7u) * per_xcd + (g >> 3);
    if (bin >= a.n_bins) return;
    const uint32_t bm_words = 1u << (a.bin_shift - 5u);
    const uint32_t n_est = 1u << (a.bin_shift - a.log2eta);
    const uint32_t k = a.k, slot = a.slot;
    const uint32_t n_words = bm_words + (n_est * k + 1u) / 2u;
    uint32_t* bm = lds;
    uint32_t* cnt = lds + bm_words;                 // 16-bit counters [estimator][slot], biased by 0x8000
    mark_runs(a, bin, lds, bm_words, n_words, list, n_list);
    // visit: bitmap word w covers the 32 cells of 16-byte chunks 2w and 2w + 1;
    // unmarked halves load the bin's first chunk instead (one line, cached),
    // so that the loads issue back to back
    uint4* chunk = reinterpret_cast<uint4*>(a.state + ((uint64_t)bin << a.bin_shift));
    const uint32_t stamp = a.stamp;
    // the listed words when they all fit the list, else every word of the bitmap
    const bool listed = n_list <= CAPPLY_LIST;
    const uint32_t n_visit = listed ? n_list : bm_words;
    // new stamps and counter moves for every chunk of a pass first, then its
    // stores; the last pass (the only one when the list holds every marked
    // word) stores after the counters, at the kernel's end, so that no wait
    // of the workgroup covers a store
    uint4 v[2 * CAPPLY_CHUNKS];
    uint32_t wd[CAPPLY_CHUNKS];
    uint32_t dirty = 0;
    for (uint32_t w0 = threadIdx.x; w0 < n_visit; w0 += blockDim.x * CAPPLY_CHUNKS) {
#pragma unroll
        for (int u = 0; u < (int)(2 * CAPPLY_CHUNKS); u++)
            if (dirty & (1u << u)) chunk[2u * wd[u / 2] + (u & 1)] = v[u];
        dirty = 0;
        uint32_t m[CAPPLY_CHUNKS];
#pragma unroll
        for (int u = 0; u < (int)CAPPLY_CHUNKS; u++) {
            const uint32_t i = w0 + (uint32_t)u * blockDim.x;
            wd[u] = i < n_visit ? (listed ? (uint32_t)list[i] : i) : 0u;
            m[u] = i < n_visit ? bm[wd[u]] : 0u;
        }
#pragma unroll
        for (int u = 0; u < (int)CAPPLY_CHUNKS; u++) {
            const uint32_t w = wd[u];
            v[2 * u] = chunk[(m[u] & 0xFFFFu) ? 2u * w : 0u];
            v[2 * u + 1] = chunk[(m[u] >> 16) ? 2u * w + 1u : 0u];
        }
#pragma unroll
        for (int u = 0; u < (int)CAPPLY_CHUNKS; u++) {
            if (!m[u]) continue;
            const uint32_t ce0 = ((wd[u] << 5) >> a.log2eta) * k;
            uint32_t changed = 0;
#pragma unroll
            for (int h = 0; h < 2; h++) {
                const uint32_t mh = (m[u] >> (16 * h)) & 0xFFFFu;
                if (!mh) continue;
                uint4& x = v[2 * u + h];
                const uint32_t before = changed;
                x.x = stamp_word(x.x, mh & 0xFu, stamp, k, slot, cnt, ce0, changed);
                x.y = stamp_word(x.y, (mh >> 4) & 0xFu, stamp, k, slot, cnt, ce0, changed);
                x.z = stamp_word(x.z, (mh >> 8) & 0xFu, stamp, k, slot, cnt, ce0, changed);
                x.w = stamp_word(x.w, (mh >> 12) & 0xFu, stamp, k, slot, cnt, ce0, changed);
                if (changed != before) dirty |= 1u << (2 * u + h);
            }
            if (changed) cnt_add(cnt, ce0 + slot, (int)changed);
        }
    }
    // every chunk load is waited for here, before any store or counter atomic
    // is in flight (a wait after them would count them too)
#pragma unroll
    for (int u = 0; u < (int)(2 * CAPPLY_CHUNKS); u++) asm volatile("" : : "v"(v[u].x), "v"(v[u].y), "v"(v[u].z), "v"(v[u].w));
    lds_barrier();
    // counters added without waiting for them (atomics whose result is unused)
    // (slot-major in memory: consecutive threads take consecutive estimators)
    uint32_t* dst = a.counts + ((uint64_t)bin << (a.bin_shift - a.log2eta));
    for (uint32_t i = threadIdx.x; i < n_est * (k + 1u); i += blockDim.x) {
        const uint32_t j = i / n_est, e = i - j * n_est;
        int c = 0;
        if (j < k) {
            const uint32_t c16 = e * k + j;
            c = (int)((cnt[c16 >> 1] >> ((c16 & 1u) * 16u)) & 0xFFFFu) - 0x8000;
        } else {
            // slot k: the estimator's live-cell total, moved by the sum of its
            // slots' moves (+1 for every cell that was not live before)
            for (uint32_t jj = 0; jj < k; jj++) {
                const uint32_t c16 = e * k + jj;
                c += (int)((cnt[c16 >> 1] >> ((c16 & 1u) * 16u)) & 0xFFFFu) - 0x8000;
            }
        }
        if (c) atomicAdd(&dst[(uint64_t)j * a.n_se + e], (uint32_t)c);
    }
#pragma unroll
    for (int u = 0; u < (int)(2 * CAPPLY_CHUNKS); u++)
        if (dirty & (1u << u)) chunk[2u * wd[u / 2] + (u & 1)] = v[u];
    // the stored values stay live to here: no register of a store in flight
    // is reused (which would wait for the store)
#pragma unroll
    for (int u = 0; u < (int)(2 * CAPPLY_CHUNKS); u++) asm volatile("" : : "v"(v[u].x), "v"(v[u].y), "v"(v[u].z), "v"(v[u].w));
}

__global__ __launch_bounds__(64 * CAPPLY_WAVES) void k_apply_counted(ApplyArgs a)
{
    extern __shared__ uint32_t lds[];
    // the marked words, in the order they were first marked
    __shared__ uint16_t list[CAPPLY_LIST];
    __shared__ uint32_t n_list;
    __shared__ uint32_t wsum[16];
    apply_counted_body(a, blockIdx.x, lds, list, n_list, wsum);
}

// Several links in one launch, as k_bin_multi (the dynamic LDS is sized for
// the largest of them).
__global__ __launch_bounds__(64 * CAPPLY_WAVES) void k_apply_counted_multi(MultiApplyArgs m)
{
    extern __shared__ uint32_t lds[];
    __shared__ uint16_t list[CAPPLY_LIST];
    __shared__ uint32_t n_list;
    __shared__ uint32_t wsum[16];
    const uint32_t l = uniform(find_link(m.wg_prefix, m.n, blockIdx.x));
    const ApplyArgs a = m.args[l];
    apply_counted_body(a, blockIdx.x - m.wg_prefix[l], lds, list, n_list, wsum);
}

// 16-bit cells (windows above 254 slots), which keep no counters: the bitmap
// stores without the counters, for calls whose offsets repeat cells.  After
// the walk a bitmap word covers 32 cells, four 16-byte chunks of eight
// cells; each chunk holding a marked cell is read once, its marked cells take
// the stamp, and it is written back if that changed it.  Unmarked chunks of a
// visited word load the bin's first chunk instead (one line, cached), so that
// the loads issue back to back.
constexpr uint32_t MARKED16_WORDS = 2;    // bitmap words per thread in flight in the visit

// Cells (two to a 32-bit word) whose bits are set in m2 take the doubled stamp s2.
__device__ __forceinline__ uint32_t restamp16(uint32_t x, uint32_t m2, uint32_t s2)
{
    const uint32_t lanes = ((m2 & 1u) ? 0x0000FFFFu : 0u) | ((m2 & 2u) ? 0xFFFF0000u : 0u);
    return (x & ~lanes) | (s2 & lanes);
}

__global__ __launch_bounds__(64 * CAPPLY_WAVES) void k_apply_marked16(ApplyArgs a)
{
    extern __shared__ uint32_t lds[];
    __shared__ uint16_t list[CAPPLY_LIST];
    __shared__ uint32_t n_list;
    const uint32_t g = blockIdx.x;
    const uint32_t per_xcd = (a.n_bins + 7u) >> 3;
    const uint32_t bin = (g & 7u) * per_xcd + (g >> 3);
    if (bin >= a.n_bins) return;
    const uint32_t bm_words = 1u << (a.bin_shift - 5u);
    mark_runs(a, bin, lds, bm_words, bm_words, list, n_list);
    uint4* chunk = reinterpret_cast<uint4*>(a.state + ((uint64_t)bin << (a.bin_shift + 1u)));    // 2 bytes a cell
    const uint32_t s2 = (a.stamp & 0xFFFFu) * 0x00010001u;
    const bool listed = n_list <= CAPPLY_LIST;
    const uint32_t n_visit = listed ? n_list : bm_words;
    for (uint32_t w0 = threadIdx.x; w0 < n_visit; w0 += blockDim.x * MARKED16_WORDS) {
        uint32_t wd[MARKED16_WORDS], m[MARKED16_WORDS];
#pragma unroll
        for (int u = 0; u < (int)MARKED16_WORDS; u++) {
            const uint32_t i = w0 + (uint32_t)u * blockDim.x;
            wd[u] = i < n_visit ? (listed ? (uint32_t)list[i] : i) : 0u;
            m[u] = i < n_visit ? lds[wd[u]] : 0u;
        }
        uint4 v[4 * MARKED16_WORDS];
#pragma unroll
        for (int u = 0; u < (int)MARKED16_WORDS; u++)
#pragma unroll
            for (int c = 0; c < 4; c++) v[4 * u + c] = chunk[((m[u] >> (8 * c)) & 0xFFu) ? 4u * wd[u] + c : 0u];
#pragma unroll
        for (int u = 0; u < (int)MARKED16_WORDS; u++) {
#pragma unroll
            for (int c = 0; c < 4; c++) {
                const uint32_t mc = (m[u] >> (8 * c)) & 0xFFu;     // cells 8c .. 8c + 7 of the word
                if (!mc) continue;
                const uint4 x = v[4 * u + c];
                uint4 y;
                y.x = restamp16(x.x, mc & 3u, s2);
                y.y = restamp16(x.y, (mc >> 2) & 3u, s2);
                y.z = restamp16(x.z, (mc >> 4) & 3u, s2);
                y.w = restamp16(x.w, (mc >> 6) & 3u, s2);
                if (y.x != x.x || y.y != x.y || y.z != x.z || y.w != x.w) chunk[4u * wd[u] + c] = y;
            }
        }
    }
}

// ---------------------------------------------------------------- hot detection
// One wave per sliding estimator: R_k = live cells (Sec. 3.2); a hot estimator
// (Sec. 3.3) sets its bit in the row bitmask and in the key-transposed bitmask;
// estimators of this slot's expiry phase clear their dead cells.  Up to CH
// 1 KiB wave loads in flight per group.

constexpr uint32_t DETECT_WAVES = 4;   // waves (estimators) per workgroup (4, 8, 16 measured: 4 best)

// R_k of estimator s and, if it is hot, its bits in the row and
// key-transposed bitmasks (lane 0 writes).
__device__ __forceinline__ void hot_mark(const LinkDesc* D, uint64_t s, uint32_t live, uint32_t lane)
{
    if (lane == 0) {
        D->rk[s] = live;
        if (live >= D->T) {
            const uint32_t q = D->q;
            const uint32_t row = (uint32_t)(s >> q), c = (uint32_t)s & ((1u << q) - 1u);
            const uint32_t sh = q - D->delta;
            const uint32_t key = c & ((1u << sh) - 1u), j = c >> sh;
            const uint32_t rw = q >= 6 ? (1u << (q - 6)) : 1u;    // words per row bitmask
            atomicOr(reinterpret_cast<unsigned long long*>(D->hotbits) + (uint64_t)row * rw + (c >> 6),
                     1ull << (c & 63u));
            atomicOr(reinterpret_cast<unsigned long long*>(D->hotT) + ((uint64_t)row * (1ull << sh) + key) * D->nw +
                         (j >> 6),
                     1ull << (j & 63u));
        }
    }
}

// The end of one estimator's test: hot_mark, and (SNAP) if hot its live-cell
// snapshot for the final test, which then reads no state.
template <bool SNAP>
__device__ __forceinline__ void hot_finish(const LinkDesc* D, uint64_t s, uint32_t live, const uint4* se, uint32_t lane)
{
    const uint32_t log2eta = D->log2eta;
    if (SNAP && live >= D->T) {
        const uint32_t chunks = 1u << (log2eta - 4);
        uint16_t* snap = D->live16 + s * chunks;
        for (uint32_t c = lane; c < chunks; c += 64u) snap[c] = (uint16_t)live_mask16(se[c], D->L);
    }
    hot_mark(D, s, live, lane);
}

// A wave covers 4 KiB of state at least: one estimator when eta >= 4096, else
// 4096 / eta consecutive estimators (load round c of the wave's four belongs
// to estimator c / (eta / 1024)), so that small estimators still give every
// wave four 1 KiB loads in flight.
// STREAM: non-temporal loads, for states that the Infinity Cache does not hold
// (1.5 GiB 334 -> 284 us, 5.7 TB/s; 320 MiB just merged into 99 -> 63 us; 24
// MiB 13 -> 15 us).
template <int CH, bool SMALL, bool STREAM>
__global__ __launch_bounds__(64 * DETECT_WAVES) void k_hot_detect(DetectArgs a)
{
    const uint32_t lane = threadIdx.x & 63u;
    const uint64_t g = (uint64_t)blockIdx.x * DETECT_WAVES + (threadIdx.x >> 6);
    // batches of up to 256 links search the wave prefix in LDS (one coalesced
    // load per workgroup instead of a chain of dependent loads per wave)
    __shared__ unsigned long long pre_lds[SMALL ? 257 : 1];
    const bool lds_prefix = SMALL && a.n_links > 1 && a.n_links <= 256u;
    if (lds_prefix) {
        for (uint32_t i = threadIdx.x; i <= a.n_links; i += blockDim.x) pre_lds[i] = a.se_prefix[i];
        __syncthreads();
    }
    if (g >= a.total) return;
    const unsigned long long* pre = lds_prefix ? pre_lds : reinterpret_cast<const unsigned long long*>(a.se_prefix);
    const uint32_t l = uniform(find_link(pre, a.n_links, g));
    const uint32_t lg = a.links[l].log2eta;
    const uint64_t s = (g - pre[l]) << (lg < 12u ? 12u - lg : 0u);      // first estimator of the wave
    const LinkDesc* D = a.links + l;
    const uint32_t log2eta = D->log2eta;
    const LiveCfg L = D->L;
    if (SMALL && log2eta < 12u) {
        // several estimators per wave: four rounds of 1 KiB, one estimator per
        // 2^(log2eta-10) rounds; every estimator is whole in this wave
        const uint32_t rpe = 1u << (log2eta - 10);       // rounds per estimator (1 or 2)
        const uint32_t ne = 4u / rpe;                    // estimators of the wave
        uint4* base = reinterpret_cast<uint4*>(D->state + (s << log2eta));
        uint4 v[4];
#pragma unroll
        for (int c = 0; c < 4; c++) v[c] = STREAM ? load_stream(base + c * 64u + lane) : base[c * 64u + lane];
        uint32_t cnt[4];
#pragma unroll
        for (int c = 0; c < 4; c++)
            cnt[c] = __popc(live_bits(v[c].x, L)) + __popc(live_bits(v[c].y, L)) + __popc(live_bits(v[c].z, L)) +
                     __popc(live_bits(v[c].w, L));
        for (uint32_t e = 0; e < ne; e++) {
            const uint64_t se_idx = s + e;
            const bool expire = (se_idx % D->expire_period) == D->expire_phase;
            uint32_t live = 0;
#pragma unroll
            for (int c = 0; c < 4; c++) {
                if ((uint32_t)c / rpe != e) continue;
                live += cnt[c];
                if (expire) {
                    uint4 n;
                    n.x = expire_word(v[c].x, L); n.y = expire_word(v[c].y, L);
                    n.z = expire_word(v[c].z, L); n.w = expire_word(v[c].w, L);
                    if (n.x != v[c].x || n.y != v[c].y || n.z != v[c].z || n.w != v[c].w) base[c * 64u + lane] = n;
                }
            }
            live = wave_sum(live);
            hot_finish<true>(D, se_idx, live, base + (uint64_t)e * rpe * 64u, lane);
        }
        return;
    }
    uint4* se = reinterpret_cast<uint4*>(D->state + (s << log2eta));
    const uint32_t per_lane = (1u << log2eta) >> 10;    // uint4 chunks per lane (eta >= 1024)
    const bool expire = (s % D->expire_period) == D->expire_phase;
    uint32_t live = 0;
    uint4 v[CH];                                        // the last group stays for the snapshot
    for (uint32_t g0 = 0; g0 < per_lane; g0 += CH) {
#pragma unroll
        for (int c = 0; c < CH; c++)
            v[c] = g0 + c >= per_lane ? make_uint4(0u, 0u, 0u, 0u)
                   : STREAM           ? load_stream(se + (g0 + c) * 64u + lane)
                                      : se[(g0 + c) * 64u + lane];
#pragma unroll
        for (int c = 0; c < CH; c++)
            if (g0 + c < per_lane)
                live += __popc(live_bits(v[c].x, L)) + __popc(live_bits(v[c].y, L)) +
                        __popc(live_bits(v[c].z, L)) + __popc(live_bits(v[c].w, L));
        if (expire) {
#pragma unroll
            for (int c = 0; c < CH; c++) {
                if (g0 + c >= per_lane) continue;
                uint4 n;
                n.x = expire_word(v[c].x, L); n.y = expire_word(v[c].y, L);
                n.z = expire_word(v[c].z, L); n.w = expire_word(v[c].w, L);
                if (n.x != v[c].x || n.y != v[c].y || n.z != v[c].z || n.w != v[c].w)
                    se[(g0 + c) * 64u + lane] = n;
            }
        }
    }
    live = wave_sum(live);
    if (per_lane <= (uint32_t)CH && live >= D->T) {
        // the whole estimator is still in registers: snapshot from there
        uint16_t* snap = D->live16 + s * (per_lane * 64u);
#pragma unroll
        for (int c = 0; c < CH; c++)
            if ((uint32_t)c < per_lane) snap[c * 64u + lane] = (uint16_t)live_mask16(v[c], L);
        hot_finish<false>(D, s, live, se, lane);
    } else {
        hot_finish<true>(D, s, live, se, lane);
    }
}

// 16-bit cells (windows above 254 slots), one link: one wave per estimator;
// in round c lane j takes the 16 cells of snapshot word c * 64 + j (two
// 16-byte chunks, so a wave reads 2 KiB in one go).  Up to CH rounds stay in
// registers for the snapshot of a hot estimator; larger estimators are read
// again.
template <int CH, bool STREAM>
__global__ __launch_bounds__(64 * DETECT_WAVES) void k_hot_detect16(DetectArgs a)
{
    const uint32_t lane = threadIdx.x & 63u;
    const uint64_t g = (uint64_t)blockIdx.x * DETECT_WAVES + (threadIdx.x >> 6);
    if (g >= a.total) return;
    const LinkDesc* D = a.links;
    const uint64_t s = g;
    const uint32_t log2eta = D->log2eta;
    const LiveCfg L = D->L;
    const uint32_t rounds = (1u << log2eta) >> 10;      // 1024 cells per wave round (eta >= 1024)
    uint4* se = reinterpret_cast<uint4*>(D->state + (s << (log2eta + 1)));
    const bool expire = (s % D->expire_period) == D->expire_phase;
    uint32_t live = 0;
    uint32_t snap[CH];
    for (uint32_t g0 = 0; g0 < rounds; g0 += CH) {
        uint4 v[2 * CH];
#pragma unroll
        for (int c = 0; c < CH; c++) {
            const uint64_t w = 2ull * ((g0 + (uint32_t)c) * 64u + lane);
            if (g0 + (uint32_t)c < rounds) {
                v[2 * c] = STREAM ? load_stream(se + w) : se[w];
                v[2 * c + 1] = STREAM ? load_stream(se + w + 1) : se[w + 1];
            }
        }
#pragma unroll
        for (int c = 0; c < CH; c++) {
            if (g0 + (uint32_t)c >= rounds) continue;
            const uint32_t m = live_mask8_c16(v[2 * c], L) | (live_mask8_c16(v[2 * c + 1], L) << 8);
            snap[c] = m;
            live += __popc(m);
            if (expire) {
                const uint64_t w = 2ull * ((g0 + (uint32_t)c) * 64u + lane);
#pragma unroll
                for (int h = 0; h < 2; h++) {
                    const uint4 x = v[2 * c + h];
                    uint4 n;
                    n.x = expire_word16(x.x, L); n.y = expire_word16(x.y, L);
                    n.z = expire_word16(x.z, L); n.w = expire_word16(x.w, L);
                    if (n.x != x.x || n.y != x.y || n.z != x.z || n.w != x.w) se[w + h] = n;
                }
            }
        }
    }
    live = wave_sum(live);
    if (live >= D->T) {
        uint16_t* out = D->live16 + s * (1u << (log2eta - 4));
        if (rounds <= (uint32_t)CH) {
#pragma unroll
            for (int c = 0; c < CH; c++)
                if ((uint32_t)c < rounds) out[c * 64u + lane] = (uint16_t)snap[c];
        } else {
            // liveness is unchanged by the expiry writes above (dead cells only)
            for (uint32_t c = 0; c < rounds; c++) {
                const uint64_t w = 2ull * (c * 64u + lane);
                out[c * 64u + lane] = (uint16_t)(live_mask8_c16(se[w], L) | (live_mask8_c16(se[w + 1], L) << 8));
            }
        }
    }
    hot_mark(D, s, live, lane);
}

// ---------------------------------------------------------------- counted detection
// R_k of every estimator from its counters (one thread per estimator): slot
// k holds the live-cell total, which every store moves by the sum of its
// moves of the per-slice slots -- the same live-cell count as a scan of the
// state, since every live cell carries the stamp of exactly one slice of the
// window.  Only the estimators that need their cells are then visited, by
// the workgroup's four waves in turn: hot ones (snapshot and bitmask bits)
// and those of this slot's expiry phase (dead cells cleared).  The slot of
// the next slice leaves the total and is zeroed for its scans.
// (workgroup blk of this link's launch; todo / todo_live / n_todo: the
// workgroup's list of estimators to visit)
__device__ __forceinline__ void count_body(const LinkDesc* D, uint64_t n_se, uint32_t blk, uint32_t* todo,
                                           uint32_t* todo_live, uint32_t& n_todo)
{
    if (threadIdx.x == 0) n_todo = 0u;
    __syncthreads();
    const uint64_t s0 = (uint64_t)blk * 256u;
    const uint64_t s = s0 + threadIdx.x;
    const uint32_t k = D->k;
    const uint32_t next = (uint32_t)((D->clock->t + 1ull) % k);
    if (s < n_se) {
        // the live-cell total (slot k) is R_k; the slot of the next slice,
        // whose cells leave the window, leaves the total and is zeroed
        const uint32_t live = D->counts[(uint64_t)k * n_se + s];
        D->counts[(uint64_t)k * n_se + s] = live - D->counts[(uint64_t)next * n_se + s];
        D->counts[(uint64_t)next * n_se + s] = 0u;
        const bool hot = live >= D->T;
        const bool expire = (s % D->expire_period) == D->expire_phase;
        if (!hot) D->rk[s] = live;
        if (hot || expire) {
            const uint32_t at = atomicAdd(&n_todo, 1u);
            todo[at] = threadIdx.x | (hot ? 0x100u : 0u) | (expire ? 0x200u : 0u);
            todo_live[at] = live;
        }
    }
    __syncthreads();
    const uint32_t wave = threadIdx.x >> 6, lane = threadIdx.x & 63u;
    const uint32_t log2eta = D->log2eta;
    const uint32_t chunks = 1u << (log2eta - 4);
    const LiveCfg L = D->L;
    for (uint32_t i = wave; i < n_todo; i += 4u) {
        const uint32_t e = todo[i];
        const uint64_t si = s0 + (e & 0xFFu);
        const bool hi = (e & 0x100u) != 0u, ei = (e & 0x200u) != 0u;
        uint4* se = reinterpret_cast<uint4*>(D->state + (si << log2eta));
        uint16_t* snap = D->live16 + si * chunks;
        // four chunks of a lane in flight (one after another: 26 against 22 us
        // for the core link's 393K counters and 6500 hot estimators)
        for (uint32_t c0 = lane; c0 < chunks; c0 += 256u) {
            uint4 v[4];
#pragma unroll
            for (uint32_t u = 0; u < 4; u++) v[u] = se[c0 + 64u * u < chunks ? c0 + 64u * u : c0];
#pragma unroll
            for (uint32_t u = 0; u < 4; u++) {
                const uint32_t c = c0 + 64u * u;
                if (c >= chunks) continue;
                if (hi) snap[c] = (uint16_t)live_mask16(v[u], L);
                if (ei) {
                    uint4 n;
                    n.x = expire_word(v[u].x, L); n.y = expire_word(v[u].y, L);
                    n.z = expire_word(v[u].z, L); n.w = expire_word(v[u].w, L);
                    if (n.x != v[u].x || n.y != v[u].y || n.z != v[u].z || n.w != v[u].w) se[c] = n;
                }
            }
        }
        if (hi) hot_finish<false>(D, si, todo_live[i], se, lane);
    }
}

__global__ __launch_bounds__(256) void k_count(const LinkDesc* link, uint64_t n_se)
{
    __shared__ uint32_t todo[256];      // local estimator | 0x100 hot | 0x200 expiring
    __shared__ uint32_t todo_live[256];
    __shared__ uint32_t n_todo;
    count_body(link, n_se, blockIdx.x, todo, todo_live, n_todo);
}

// Several counted links of an engine in one launch: workgroup g works for
// link ids[l] with wg_prefix[l] <= g < wg_prefix[l + 1].
__global__ __launch_bounds__(256) void k_count_multi(CountMultiArgs m)
{
    __shared__ uint32_t todo[256];
    __shared__ uint32_t todo_live[256];
    __shared__ uint32_t n_todo;
    const uint32_t l = uniform(find_link(m.wg_prefix, m.n, blockIdx.x));
    const LinkDesc* D = m.links + m.ids[l];
    count_body(D, D->n_se, blockIdx.x - m.wg_prefix[l], todo, todo_live, n_todo);
}

// Bytes of a word equal to stamp s.
__device__ __forceinline__ uint32_t count_eq(uint32_t w, uint32_t s)
{
    const uint32_t x = w ^ (s * 0x01010101u);
    const uint32_t nz = (((x & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | x) & 0x80808080u;
    return 4u - __popc(nz);
}

// The per-slot counters rebuilt from the state (one wave per estimator): for
// every slice of the window, the cells holding its stamp.
__global__ __launch_bounds__(256) void k_recount(const LinkDesc* link, uint64_t n_se)
{
    const LinkDesc* D = link;
    const uint64_t s = (uint64_t)blockIdx.x * 4u + (threadIdx.x >> 6);
    const uint32_t lane = threadIdx.x & 63u;
    if (s >= n_se) return;
    const uint32_t k = D->k;
    const unsigned long long t = D->clock->t;
    const uint32_t slot = (uint32_t)(t % k);
    const uint32_t chunks = 1u << (D->log2eta - 4);
    const uint4* se = reinterpret_cast<const uint4*>(D->state + (s << D->log2eta));
    uint32_t total = 0;
    for (uint32_t j = 0; j < k; j++) {
        const uint32_t d = slot >= j ? slot - j : slot + k - j;   // slices back from t
        uint32_t n = 0;
        if (d <= t) {
            const uint32_t st = 1u + (uint32_t)((t - d) % 255ull);
            for (uint32_t c = lane; c < chunks; c += 64u) {
                const uint4 v = se[c];
                n += count_eq(v.x, st) + count_eq(v.y, st) + count_eq(v.z, st) + count_eq(v.w, st);
            }
        }
        n = wave_sum(n);
        total += n;
        if (lane == 0) D->counts[(uint64_t)j * n_se + s] = n;
    }
    if (lane == 0) D->counts[(uint64_t)k * n_se + s] = total;      // the live-cell total
}

// ---------------------------------------------------------------- hot lists
// One 1024-thread block per (link, row): the ascending list of hot columns,
// from the row bitmask.  The row-0 block also clears the link's counters.

__global__ __launch_bounds__(1024) void k_hot_compact(const LinkDesc* links, const uint32_t* row_table)
{
    __shared__ uint32_t lds[16];
    const uint32_t rt = row_table[blockIdx.x];
    const LinkDesc* D = links + (rt >> 8);
    const uint32_t row = rt & 255u;
    const uint32_t q = D->q;
    const uint32_t words = q >= 6 ? (1u << (q - 6)) : 1u;
    const uint64_t* bits = D->hotbits + (uint64_t)row * words;
    if (row == 0 && threadIdx.x == 0) {
        for (int l = 0; l < (int)MAX_ROWS; l++) D->ctl->level_n[l] = 0;
        D->ctl->n_acc = 0;
        D->ctl->n_out = 0;
    }
    const uint32_t per = (words + 1023u) / 1024u;
    const uint32_t w0 = min(words, threadIdx.x * per), w1 = min(words, w0 + per);
    uint32_t cnt = 0;
    for (uint32_t w = w0; w < w1; w++) cnt += __popcll(bits[w]);
    uint32_t total;
    uint32_t off = block_exclusive_scan_1024(cnt, lds, &total);
    uint32_t* list = D->hot_list + ((uint64_t)row << q);
    for (uint32_t w = w0; w < w1; w++) {
        uint64_t b = bits[w];
        while (b) {
            const uint32_t i = (uint32_t)__ffsll((long long)b) - 1u;
            b &= b - 1;
            list[off++] = w * 64u + i;
        }
    }
    if (threadIdx.x == 0) D->ctl->hot_n[row] = total;
}

// ---------------------------------------------------------------- level work
// Work items of one level for every link, prefix-summed; expansion levels pad
// each link to whole 256-item blocks so that a block never spans two links.

// log2 of the lanes that test one tuple: 128 cells of an estimator each (eta
// >= 1024), at most a wave.
__device__ __forceinline__ uint32_t verify_lanes_log2(uint32_t log2eta) { return min(6u, log2eta - 7u); }

// Work items of one link at a level: 0 = |HSE(0)| x |HSE(1)| pairs of rows
// 0, 1; L = the tuples of level L-1 (extended by row L+2); LEVEL_DFS = waves'
// worth of pairs of rows 0, 1 (extended over all rows); LEVEL_VERIFY = the
// waves' worth of full tuples.  The items of levels 0 and L are padded to
// whole 256-item workgroups, so a workgroup never spans two links and appends
// with one atomic.
__device__ __forceinline__ unsigned long long level_items(const LinkDesc* D, uint32_t level)
{
    const Ctl* c = D->ctl;
    unsigned long long n = 0;
    if (level == 0) {
        n = (unsigned long long)c->hot_n[0] * c->hot_n[1];
    } else if (level == LEVEL_DFS) {
        // a wave takes 64 pairs
        return ((unsigned long long)c->hot_n[0] * c->hot_n[1] + 63ull) >> 6;
    } else if (level == LEVEL_VERIFY) {
        // a wave takes 64 / (lanes per tuple) tuples at a time
        const unsigned long long m = c->level_n[D->r - 3];
        const uint32_t sh = 6u - verify_lanes_log2(D->log2eta);
        return ((m < D->max_tuples ? m : D->max_tuples) + (1ull << sh) - 1ull) >> sh;
    } else if (level + 2 < D->r) {
        const unsigned long long m = c->level_n[level - 1];
        n = m < D->max_tuples ? m : D->max_tuples;
    }
    return (n + 255ull) & ~255ull;
}

// Every workgroup (of at least 256 threads) of a level kernel computes the
// level's prefix of work items over the links into LDS (pre[0..n_links]) from
// the counters the previous kernel left: no separate launch between levels.
__device__ void level_prefix_lds(const LevelArgs& a, unsigned long long* pre)
{
    __shared__ unsigned long long part[256];
    if (a.n_links == 1) {
        if (threadIdx.x == 0) {
            pre[0] = 0;
            pre[1] = level_items(a.links, a.level);
        }
        __syncthreads();
        return;
    }
    const bool in = threadIdx.x < 256u;
    const uint32_t per = (a.n_links + 255u) / 256u;
    const uint32_t l0 = in ? min(a.n_links, threadIdx.x * per) : a.n_links, l1 = min(a.n_links, l0 + per);
    unsigned long long sum = 0;
    for (uint32_t l = l0; l < l1; l++) {
        const unsigned long long n = level_items(a.links + l, a.level);
        pre[l] = n;
        sum += n;
    }
    if (in) part[threadIdx.x] = sum;
    __syncthreads();
    for (uint32_t o = 1; o < 256u; o <<= 1) {
        const unsigned long long v = in && threadIdx.x >= o ? part[threadIdx.x - o] : 0ull;
        __syncthreads();
        if (in) part[threadIdx.x] += v;
        __syncthreads();
    }
    unsigned long long run = in ? part[threadIdx.x] - sum : 0ull;
    for (uint32_t l = l0; l < l1; l++) {
        const unsigned long long n = pre[l];
        pre[l] = run;
        run += n;
    }
    if (threadIdx.x == 255u) pre[a.n_links] = part[255];
    __syncthreads();
}

// ---------------------------------------------------------------- expansion
// Sec. 4.2, with the cross products of Alg. 6/7 replaced by a lookup: for a
// tuple with he_0 and he_{i-1}, the overlap test fixes the low q-delta bits of
// he_i, so the candidates are exactly the hot columns of row i under that key
// (one transposed bitmask word per 64 candidates).  A tuple is stored as
// (he_0, x) with x the host bits regained so far; he_i = (x >> (i-1)delta) mod
// 2^q XOR he_0.  Tuples are appended with one atomic per block; their order is
// not deterministic, the set is.

template <bool EMIT>
__device__ __forceinline__ uint32_t extend_one(const LinkDesc* D, uint32_t he0, uint64_t x, uint32_t row,
                                               uint64_t* out_x, uint32_t* out_h0, uint64_t slot, uint32_t valid)
{
    if (!valid) return 0;
    const uint32_t q = D->q, delta = D->delta, nw = D->nw, key_bits = D->key_bits;
    const uint32_t qmask = (1u << q) - 1u;
    const uint32_t sh = q - delta;
    const uint32_t kmask = (1u << sh) - 1u;
    const uint32_t bprev = (uint32_t)(x >> ((row - 2) * delta)) & qmask;       // B(row-1)
    const uint32_t key = ((bprev >> delta) ^ he0) & kmask;
    const uint64_t* w = D->hotT + ((uint64_t)row * (1ull << sh) + key) * nw;
    const uint32_t newpos = (row - 2) * delta + q;           // first host bit B(row) adds
    const uint32_t dmask = (1u << delta) - 1u;
    const uint32_t top0 = he0 >> sh;
    const uint64_t cap = D->max_tuples;
    uint32_t cnt = 0;
    for (uint32_t wi = 0; wi < nw; wi++) {
        uint64_t bits = w[wi];
        while (bits) {
            const uint32_t j = (uint32_t)__ffsll((long long)bits) - 1u + wi * 64u;
            bits &= bits - 1;
            const uint64_t v = (uint64_t)((top0 ^ j) & dmask);              // top delta bits of B(row)
            const uint64_t nx = x | (v << newpos);
            if ((nx >> key_bits) != 0) continue;                           // bits beyond the key width
            if (EMIT) {
                if (slot + cnt < cap) {
                    out_x[slot + cnt] = nx;
                    out_h0[slot + cnt] = he0;
                }
            }
            cnt++;
        }
    }
    return cnt;
}

// Level 0: every (he_0, he_1) from HSE(0) x HSE(1), extended over row 2.
__global__ __launch_bounds__(256) void k_expand0(LevelArgs a)
{
    extern __shared__ unsigned long long pre[];      // [n_links + 1], sized at launch
    level_prefix_lds(a, pre);
    const uint64_t total = pre[a.n_links];
    for (uint64_t base = (uint64_t)blockIdx.x * 256u; base < total; base += (uint64_t)gridDim.x * 256u) {
        const uint32_t l = uniform(find_link(pre, a.n_links, base));
        const LinkDesc* D = a.links + l;
        const uint64_t n0 = D->ctl->hot_n[0], n1 = D->ctl->hot_n[1];
        const uint64_t Q = n0 * n1;
        const uint64_t idx = base - pre[l] + threadIdx.x;
        const uint32_t qmask = (1u << D->q) - 1u;
        uint32_t ok = idx < Q;
        uint32_t he0 = 0;
        uint64_t x = 0;
        if (ok) {
            uint64_t ia, ib;
            if (Q <= 0xFFFFFFFFull) { ia = (uint32_t)idx / (uint32_t)n1; ib = (uint32_t)idx - (uint32_t)ia * (uint32_t)n1; }
            else { ia = idx / n1; ib = idx % n1; }
            he0 = D->hot_list[ia];
            const uint32_t he1 = D->hot_list[(1ull << D->q) + ib];
            x = (uint64_t)((he0 ^ he1) & qmask);                 // B(1): host bits 0..q-1
            if ((x >> D->key_bits) != 0) ok = 0;
        }
        uint64_t* ox = D->ctb_x[0];
        uint32_t* oh = D->ctb_h0[0];
        const uint32_t cnt = extend_one<false>(D, he0, x, 2, ox, oh, 0, ok);
        const unsigned long long slot = block_append_256(cnt, &D->ctl->level_n[0]);
        extend_one<true>(D, he0, x, 2, ox, oh, slot, ok);
    }
}

// Level L >= 1: extend the tuples of level L-1 over row L+2.
__global__ __launch_bounds__(256) void k_extend(LevelArgs a)
{
    extern __shared__ unsigned long long pre[];      // [n_links + 1], sized at launch
    level_prefix_lds(a, pre);
    const uint32_t level = a.level, row = level + 2;
    const uint64_t total = pre[a.n_links];
    for (uint64_t base = (uint64_t)blockIdx.x * 256u; base < total; base += (uint64_t)gridDim.x * 256u) {
        const uint32_t l = uniform(find_link(pre, a.n_links, base));
        const LinkDesc* D = a.links + l;
        const unsigned long long raw = D->ctl->level_n[level - 1];
        const uint64_t nin = raw < D->max_tuples ? raw : D->max_tuples;
        const uint64_t idx = base - pre[l] + threadIdx.x;
        const uint32_t valid = idx < nin;
        const uint64_t* ix = D->ctb_x[(level - 1) & 1];
        const uint32_t* ih = D->ctb_h0[(level - 1) & 1];
        const uint32_t he0 = valid ? ih[idx] : 0u;
        const uint64_t x = valid ? ix[idx] : 0ull;
        uint64_t* ox = D->ctb_x[level & 1];
        uint32_t* oh = D->ctb_h0[level & 1];
        const uint32_t cnt = extend_one<false>(D, he0, x, row, ox, oh, 0, valid);
        const unsigned long long slot = block_append_256(cnt, &D->ctl->level_n[level]);
        extend_one<true>(D, he0, x, row, ox, oh, slot, valid);
    }
}

// ---------------------------------------------------------------- depth-first expansion
// The same candidate tuples as the level-by-level kernels above, in one
// launch.  Every level's tuple count still goes to level_n (capacity checks
// and diagnostics); the order of the tuples is not deterministic.
//
// Few of the |HSE(0)| x |HSE(1)| pairs extend, and those unevenly, so a
// thread per pair leaves most lanes of a wave idle, and nested loops over the
// rows step through the product of its lanes' longest rows.  Here every wave
// keeps a queue per row in LDS, of partial tuples with candidates of that row
// left, and each of its steps works for up to 64 of them:
//   - 64 pairs at a time, far apart in the list of pairs (a host's estimators
//     extend in bulk, its neighbours not at all), are looked up; those with
//     candidates of row 2 enter its queue;
//   - a step takes the 64 newest partial tuples of the deepest row that has
//     64, and of each its next candidate: the extended tuple enters the next
//     row's queue (or, after the last row, the output), the tuple itself goes
//     back while it has candidates left.  So no queue ever holds more than
//     127, and the lanes are full until the end.
// All lookups go to LDS: the hot bits of rows 2..r-1, 2^q per row in key order
// (bit (key << delta) + j), and the hot columns of rows 0 and 1.  (Workgroups
// with few pairs of a link read its hot bits where they are: filling LDS with
// them is most of their time.  24 links of few hot columns 19.3 us with every
// table filled, 12.0 so, 64 links of many 52 and 45.)  The walk
// counts the tuples and keeps a wave's first DFS_OUT full ones in LDS; the
// workgroup then reserves its slots with one atomic, and a wave with more
// tuples walks again to write them (atomics of one address pass at about 12 ns
// each: appending 192 tuples at a time took 84 us for 1.4M of them).  For
// delta <= 6 (one 64-bit word of candidates a key) and links whose hot bits
// leave room for the queues; others take the nested walk of k_expand_nested.

// A wave's view of the link it expands.
struct DfsLink {
    const uint32_t* tab;              // packed hot bits of rows 2.. (short runs: not filled)
    const uint64_t* keys;             // the same in memory, a word a key
    uint4* queue;                     // [r - 2][DFS_QUEUE]: x, he_0, candidates left
    uint2* out;                       // [DFS_OUT]: the wave's first full tuples (x, he_0)
    uint64_t* out_x;
    uint32_t* out_h0;
    uint64_t max_tuples;
    uint32_t words, delta, sh, kmask, qmask, key_bits, r;
    bool in_lds;
};

// Orders a wave's LDS accesses across its lanes.
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ uint32_t lanes_below(uint64_t mask)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// The candidates of `row` under a key, as a word of up to 2^6 bits.
__device__ __forceinline__ uint64_t dfs_candidates(const DfsLink& d, uint32_t row, uint32_t key)
{
    if (!d.in_lds) return d.keys[((uint64_t)row << d.sh) + key];
    const uint32_t bit = key << d.delta;
    const uint32_t* w = d.tab + (row - 2u) * d.words + (bit >> 5);
    if (d.delta == 6u) return (uint64_t)w[1] << 32 | w[0];
    if (d.delta == 5u) return w[0];
    return (w[0] >> (bit & 31u)) & ((1u << (1u << d.delta)) - 1u);
}

// The packed hot bits of rows 2..r-1 of link D (delta <= 6) into LDS.
__device__ __forceinline__ void load_hot_table(const LinkDesc* D, uint32_t words, uint32_t* tab)
{
    const uint32_t delta = D->delta, sh = D->q - delta, n = (D->r - 2u) * words;
    const uint32_t lg = 31u - (uint32_t)__clz((int)words);
    const uint32_t* src = reinterpret_cast<const uint32_t*>(D->hotT);
    for (uint32_t i = threadIdx.x; i < n; i += blockDim.x) {
        const uint32_t row = 2u + (i >> lg), w = i & (words - 1u);       // words per row: a power of two
        uint32_t v = 0;
        if (delta == 6u) {
            v = src[(uint64_t)row * words + w];              // a 64-bit word a key: the same order
        } else {
            // one 64-bit word a key, its low 2^delta bits in use
            const uint32_t key0 = (w << 5) >> delta, keys = min(32u >> delta, 1u << sh);
            for (uint32_t m = 0; m < keys; m++)
                v |= src[2u * (((uint64_t)row << sh) + key0 + m)] << (m << delta);
        }
        tab[i] = v;
    }
}

// A wave's walk over its work items it, it + step, .. below `end` of n_items:
// item i is the pairs i + lane * n_items of n0 x n1.  The tuples accepted per
// level are added to lv (LDS, this wave's) and the first DFS_OUT full ones
// staged; with `emit` the full ones go to slot, slot + 1, .. instead.  One loop, one copy of the step
// whatever the row: a close runs this code once, so every cache line of it is
// fetched cold (the step unrolled over the rows, in both walks, took 15 us
// where there was next to nothing to expand).
__device__ __forceinline__ void dfs_walk(const DfsLink& d, const uint32_t* l0, const uint32_t* l1, uint32_t n0,
                                         uint32_t n1, uint64_t n_items, uint64_t it, uint64_t step, uint64_t end,
                                         uint32_t* lv, bool emit, uint64_t slot)
{
    const uint64_t Q = (uint64_t)n0 * n1;
    const uint32_t lane = threadIdx.x & 63u;
    uint64_t cnt = 0;                   // the queues' sizes (at most 127), a byte each, from row 2's up
    for (;;) {
        // the newest entries of the deepest row that fills the wave; else new
        // pairs; else the first row with any (what it adds fills the others)
        const uint64_t full = cnt & 0x4040404040404040ull;
        uint32_t level, x = 0, he0 = 0, next = 2;
        uint64_t c = 0;                 // candidates of row `next` of the tuple (he0, x)
        if (!full && it < end) {
            const uint64_t p = it + lane * n_items;
            it += step;
            level = ~0u;
            if (p < Q) {
                const uint32_t ia = Q <= 0xFFFFFFFFull ? (uint32_t)p / n1 : (uint32_t)(p / n1);
                he0 = l0[ia];
                x = (he0 ^ l1[(uint32_t)(p - (uint64_t)ia * n1)]) & d.qmask;     // B(1): host bits 0..q-1
                if (d.key_bits >= 32u || (x >> d.key_bits) == 0u) c = 1ull;
            }
        } else {
            if (!cnt) break;
            level = (full ? 63u - (uint32_t)__clzll((long long)full) : (uint32_t)__ffsll((long long)cnt) - 1u) >> 3;
            const uint32_t row = level + 2u, n = (uint32_t)(cnt >> (8u * level)) & 0xFFu;
            const uint32_t m = min(64u, n), base = n - m;
            uint4* q = d.queue + level * DFS_QUEUE;
            const bool in = lane < m;
            uint4 t = make_uint4(0u, 0u, 0u, 0u);
            if (in) t = q[base + lane];
            wave_sync();
            he0 = t.y;
            uint64_t bits = (uint64_t)t.w << 32 | t.z;
            const uint32_t j = (uint32_t)__ffsll((long long)bits) - 1u;
            bits &= bits - 1ull;
            // back while candidates are left
            const uint64_t back = __ballot(in && bits != 0ull);
            if (in && bits != 0ull) q[base + lanes_below(back)] = make_uint4(t.x, he0, (uint32_t)bits, (uint32_t)(bits >> 32));
            cnt -= (uint64_t)(m - (uint32_t)__popcll(back)) << (8u * level);
            // the top delta bits of B(row), host bits pos..; none may lie beyond the key width
            const uint32_t pos = (row - 1u) * d.delta + d.sh;
            const uint32_t v = ((he0 >> d.sh) ^ j) & ((1u << d.delta) - 1u);
            const bool ok = in && (d.key_bits >= pos + d.delta || (v >> (d.key_bits > pos ? d.key_bits - pos : 0u)) == 0u);
            x = pos < 32u ? t.x | (v << pos) : t.x;
            const uint64_t good = __ballot(ok);
            next = row + 1u;
            c = ok ? 1ull : 0ull;
            if (!emit && lane == 0) lv[level] += (uint32_t)__popcll(good);
            if (next == d.r) {
                const uint64_t at = slot + lanes_below(good);
                if (ok && !emit && at < DFS_OUT) d.out[at] = make_uint2(x, he0);
                if (ok && emit && at < d.max_tuples) {
                    d.out_x[at] = x;
                    d.out_h0[at] = he0;
                }
                slot += (uint64_t)__popcll(good);
            }
        }
        if (next < d.r) {
            if (c) c = dfs_candidates(d, next, ((((x >> ((next - 2u) * d.delta)) & d.qmask) >> d.delta) ^ he0) & d.kmask);
            const uint64_t on = __ballot(c != 0ull);
            const uint32_t sh = 8u * (next - 2u);
            if (c) d.queue[(next - 2u) * DFS_QUEUE + ((uint32_t)(cnt >> sh) & 0xFFu) + lanes_below(on)] =
                       make_uint4(x, he0, (uint32_t)c, (uint32_t)(c >> 32));
            cnt += (uint64_t)__popcll(on) << sh;
        }
        wave_sync();
    }
}

// One link's items are dealt to all waves in turn; several links' in
// contiguous runs per workgroup, so that it meets few links and loads few
// tables: none for a run of at most DFS_LOOKUP_ITEMS items a wave (64 links:
// 52 us with every table loaded, 46 at 1 and 2, 45 at 4 and at 16).  A link
// alone loads its table for more items a wave than the table has times
// DFS_LOOKUP_WORDS words (of six rows of 2^16 columns 16: 3 hot columns a row
// 16.2 us with the table and 9.1 looked up, 1300 28.6 and 19; of 2^12 columns
// 1: 30 hot columns 12.2 and 12.5).
constexpr uint32_t DFS_LOOKUP_ITEMS = 4, DFS_LOOKUP_WORDS = 512;
template <int LEVELS, uint32_t WAVES>
__global__ __launch_bounds__(64 * WAVES) void k_expand_dfs(LevelArgs a)
{
    // [n_links + 1] prefix; per wave the queues and the staged tuples; hot
    // columns of rows 0 and 1; packed hot bits
    extern __shared__ __align__(16) unsigned long long pre[];
    __shared__ uint32_t lv_wave[WAVES][LEVELS];
    __shared__ unsigned long long out_base;
    const uint32_t lane = threadIdx.x & 63u, wid = threadIdx.x >> 6;
    const bool one = a.n_links == 1u;
    if (!one) level_prefix_lds(a, pre);
    uint4* queues = reinterpret_cast<uint4*>(pre + ((a.n_links + 2u) & ~1u));
    uint2* outs = reinterpret_cast<uint2*>(queues + WAVES * a.queue_rows * DFS_QUEUE);
    uint32_t* lists = reinterpret_cast<uint32_t*>(outs + WAVES * DFS_OUT);
    uint32_t* tab = lists + 2u * DFS_LIST;
    const uint64_t n_items = one ? level_items(a.links, LEVEL_DFS) : pre[a.n_links];
    uint64_t item = one ? 0u : n_items * blockIdx.x / gridDim.x;
    const uint64_t end = one ? n_items : n_items * (blockIdx.x + 1ull) / gridDim.x;
    if (one && (uint64_t)blockIdx.x >= n_items) return;
    while (item < end) {
        // the run of this workgroup's items that belong to one link
        const uint32_t l = one ? 0u : uniform(find_link(pre, a.n_links, item));
        const LinkDesc* D = a.links + l;
        const uint64_t link0 = one ? 0ull : pre[l], link_items = (one ? n_items : pre[l + 1]) - link0;
        const uint64_t run_end = min(link0 + link_items, end);
        const uint32_t n0 = D->ctl->hot_n[0], n1 = D->ctl->hot_n[1], lf = D->r - 3u;
        DfsLink d;
        d.delta = D->delta; d.sh = D->q - d.delta; d.r = D->r; d.key_bits = D->key_bits;
        d.kmask = (1u << d.sh) - 1u;
        d.qmask = (1u << D->q) - 1u;
        d.words = dfs_row_words(D->q);
        d.max_tuples = D->max_tuples;
        d.out_x = D->ctb_x[lf & 1u];
        d.out_h0 = D->ctb_h0[lf & 1u];
        d.tab = tab;
        d.keys = D->hotT;
        d.in_lds = one ? n_items > (uint64_t)gridDim.x * WAVES * ((d.r - 2u) * d.words / DFS_LOOKUP_WORDS)
                       : run_end - item > (uint64_t)DFS_LOOKUP_ITEMS * WAVES;
        d.queue = queues + wid * a.queue_rows * DFS_QUEUE;
        d.out = outs + wid * DFS_OUT;
        const uint32_t *l0 = D->hot_list, *l1 = D->hot_list + (1ull << D->q);
        if (lane < (uint32_t)LEVELS) lv_wave[wid][lane] = 0u;
        if (n0 <= DFS_LIST && n1 <= DFS_LIST) {          // (longer lists are read where they are)
            const uint32_t n = max(n0, n1);
            for (uint32_t i = threadIdx.x; i < n; i += 64u * WAVES) {
                const uint32_t c0 = l0[min(i, n0 - 1u)], c1 = l1[min(i, n1 - 1u)];
                lists[i] = c0;
                lists[DFS_LIST + i] = c1;
            }
            l0 = lists;
            l1 = lists + DFS_LIST;
        }
        if (d.in_lds) load_hot_table(D, d.words, tab);
        __syncthreads();
        const uint64_t it = one ? (uint64_t)wid * gridDim.x + blockIdx.x : item - link0 + wid;
        const uint64_t step = one ? (uint64_t)gridDim.x * WAVES : WAVES, it_end = run_end - link0;
        uint64_t slot = 0;
        for (uint32_t pass = 0; pass < 2u; pass++) {
            const uint32_t mine = lv_wave[wid][lf];          // the wave's full tuples, once counted
            if (pass && mine <= DFS_OUT) {
                for (uint32_t i = lane; i < mine; i += 64u) {
                    const uint2 v = d.out[i];
                    if (slot + i < d.max_tuples) {
                        d.out_x[slot + i] = v.x;
                        d.out_h0[slot + i] = v.y;
                    }
                }
            } else if (!pass || slot < d.max_tuples) {
                dfs_walk(d, l0, l1, n0, n1, link_items, it, step, it_end, lv_wave[wid], pass != 0u, slot);
            }
            __syncthreads();
            if (pass) break;
            if (threadIdx.x <= lf) {
                unsigned long long v = 0;
                for (uint32_t w = 0; w < WAVES; w++) v += lv_wave[w][threadIdx.x];
                const unsigned long long at = v ? atomicAdd(&D->ctl->level_n[threadIdx.x], v) : 0ull;
                if (threadIdx.x == lf) out_base = at;
            }
            __syncthreads();
            slot = out_base;
            for (uint32_t w = 0; w < wid; w++) slot += lv_wave[w][lf];
        }
        item = run_end;
    }
}

// Level-0 pair idx of n0 x n1: (he0, B(1)); false if idx is padding or B(1)
// has bits beyond the key width.
__device__ __forceinline__ bool level0_pair(const LinkDesc* D, uint64_t idx, uint32_t* he0, uint64_t* x)
{
    const uint64_t n0 = D->ctl->hot_n[0], n1 = D->ctl->hot_n[1];
    const uint64_t Q = n0 * n1;
    if (idx >= Q) return false;
    uint64_t ia, ib;
    if (Q <= 0xFFFFFFFFull) { ia = (uint32_t)idx / (uint32_t)n1; ib = (uint32_t)idx - (uint32_t)ia * (uint32_t)n1; }
    else { ia = idx / n1; ib = idx % n1; }
    *he0 = D->hot_list[ia];
    const uint32_t he1 = D->hot_list[(1ull << D->q) + ib];
    *x = (uint64_t)((*he0 ^ he1) & ((1u << D->q) - 1u));                 // B(1): host bits 0..q-1
    return (*x >> D->key_bits) == 0;
}

// The nested walk, with the hot bits in memory: rows are template levels, so
// the loop state of every row lives in registers; each thread takes pairs of
// HSE(0) x HSE(1).  A count pass reserves the workgroup's slots in the
// full-tuple buffer, a second pass writes them.
template <int RMAX>
struct DfsCtx {
    uint32_t lv[RMAX];            // tuples accepted per level, this thread
    uint64_t slot;                // write pass: this thread's next slot
    uint64_t* out_x;
    uint32_t* out_h0;
};

// rows ROW..r-1 still to choose (r <= RMAX, a compile-time bound that keeps
// every row's loop state in registers)
template <int ROW, int RMAX, bool EMIT>
__device__ __forceinline__ void dfs_row(const LinkDesc* D, uint32_t he0, uint64_t x, DfsCtx<RMAX>& c)
{
    if (ROW == RMAX || (uint32_t)ROW >= D->r) {             // rows 0..r-1 all chosen: a full tuple
        if (EMIT) {
            if (c.slot < D->max_tuples) {
                c.out_x[c.slot] = x;
                c.out_h0[c.slot] = he0;
            }
            c.slot++;
        }
        return;
    }
    if constexpr (ROW < RMAX) {
        const uint32_t q = D->q, delta = D->delta, nw = D->nw, key_bits = D->key_bits;
        const uint32_t qmask = (1u << q) - 1u;
        const uint32_t sh = q - delta;
        const uint32_t bprev = (uint32_t)(x >> ((ROW - 2) * delta)) & qmask;     // B(ROW-1)
        const uint32_t key = ((bprev >> delta) ^ he0) & ((1u << sh) - 1u);
        const uint64_t* w = D->hotT + ((uint64_t)ROW * (1ull << sh) + key) * nw;
        const uint32_t newpos = (ROW - 2) * delta + q;                           // first host bit B(ROW) adds
        const uint32_t top0 = he0 >> sh;
        for (uint32_t wi = 0; wi < nw; wi++) {
            uint64_t bits = w[wi];
            while (bits) {
                const uint32_t j = (uint32_t)__ffsll((long long)bits) - 1u + wi * 64u;
                bits &= bits - 1;
                const uint64_t nx = x | ((uint64_t)((top0 ^ j) & ((1u << delta) - 1u)) << newpos);
                if ((nx >> key_bits) != 0) continue;                              // bits beyond the key width
                c.lv[ROW - 2]++;
                dfs_row<ROW + 1, RMAX, EMIT>(D, he0, nx, c);
            }
        }
    }
}

// A workgroup's slots for its threads' tuples of one link: the totals per
// level to level_n, and this thread's first full-tuple slot (base of the
// workgroup, then the tuples of the lanes and waves before it).  lv: tuples
// per level (the last one are the full ones, *n_full).  All threads call it.
template <int RMAX>
__device__ __forceinline__ uint64_t reserve_tuples(const LinkDesc* D, const uint32_t* lv, uint32_t (*wsum)[RMAX],
                                                   unsigned long long* base_slot, uint32_t* n_full)
{
    const uint32_t lane = threadIdx.x & 63u, wid = threadIdx.x >> 6;
    const uint32_t r = D->r, lf = r - 3;
    uint32_t full = 0;
#pragma unroll
    for (uint32_t L = 0; L + 2 < (uint32_t)RMAX; L++) {
        if (L == lf) full = lv[L];
        const uint32_t v = wave_sum(L <= lf ? lv[L] : 0u);
        if (lane == 0) wsum[wid][L] = v;
    }
    uint32_t incl = full;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t v = __shfl_up(incl, o, 64);
        if (lane >= (uint32_t)o) incl += v;
    }
    __syncthreads();
    if (threadIdx.x <= lf) {
        const uint32_t L = threadIdx.x;
        unsigned long long v = 0;
        for (uint32_t w = 0; w < 4u; w++) v += wsum[w][L];
        const unsigned long long at = v ? atomicAdd(&D->ctl->level_n[L], v) : 0ull;
        if (L == lf) *base_slot = at;
    }
    __syncthreads();
    uint64_t before = 0;
    for (uint32_t w = 0; w < wid; w++) before += wsum[w][lf];
    *n_full = full;
    return *base_slot + before + (incl - full);
}

template <int RMAX>
__global__ __launch_bounds__(256) void k_expand_nested(LevelArgs a)
{
    extern __shared__ unsigned long long pre[];      // [n_links + 1], sized at launch
    __shared__ uint32_t wsum[4][RMAX];
    __shared__ unsigned long long base_slot;
    level_prefix_lds(a, pre);
    const uint64_t n_chunks = pre[a.n_links] / 256u;
    uint64_t chunk = blockIdx.x;
    while (chunk < n_chunks) {
        // the run of this workgroup's chunks that belong to one link
        const uint32_t l = uniform(find_link(pre, a.n_links, chunk * 256u));
        const LinkDesc* D = a.links + l;
        const uint64_t link_end = pre[l + 1] / 256u;
        DfsCtx<RMAX> c{};
        c.out_x = D->ctb_x[(D->r - 3u) & 1u];
        c.out_h0 = D->ctb_h0[(D->r - 3u) & 1u];
        uint64_t ch = chunk;
        for (; ch < link_end; ch += gridDim.x) {
            uint32_t he0;
            uint64_t x;
            if (level0_pair(D, ch * 256u - pre[l] + threadIdx.x, &he0, &x)) dfs_row<2, RMAX, false>(D, he0, x, c);
        }
        uint32_t full;
        c.slot = reserve_tuples<RMAX>(D, c.lv, wsum, &base_slot, &full);
        // (most threads have none to write: 2000 hosts into 2^17 columns 342 us with
        // the second walk by all, 252 so; nor is there room past the buffer)
        const bool writes = full && c.slot < D->max_tuples;
        for (uint64_t cw = chunk; writes && cw < link_end; cw += gridDim.x) {
            uint32_t he0;
            uint64_t x;
            if (level0_pair(D, cw * 256u - pre[l] + threadIdx.x, &he0, &x)) dfs_row<2, RMAX, true>(D, he0, x, c);
        }
        __syncthreads();
        chunk = ch;
    }
}

// ---------------------------------------------------------------- verify
// Final test of every full tuple (end of Alg. 4, Sec. 4.2 last pass): optional
// re-hash check, then the UnionSE of Alg. 1 -- a cell counts only when it is
// live in all r estimators -- and R >= T.
//
// Bound by the L2 reads of the live-cell snapshots.  eta / 128 lanes take a
// tuple (one 16-byte load per row), so a wave tests 64 / lanes consecutive
// tuples at a time: at eta = 2048 four, where a wave per tuple left half its
// lanes idle and made 32 8-byte loads per row.  A union's count only falls
// with every row, so the first three rows are counted first and the others
// are read only for tuples that can still reach T: most false tuples cannot.

//
// One link's accepted keys are collected in LDS and appended once per
// workgroup: atomics of one address pass at about 12 ns each, 12 us for the
// 1000 hosts of a small close (several links append to a counter each).
// Measured against a wave and five full rows per tuple: 1.4M tuples at eta =
// 2048, r = 5 508 -> 131 us (13.7 TB/s of snapshots); 6000 tuples with 1000
// accepted at eta = 1024, r = 6 17 -> 10 us.

constexpr uint32_t VERIFY_THREADS = 1024, VERIFY_LIST = 1024;

__global__ __launch_bounds__(VERIFY_THREADS) void k_verify(LevelArgs a)
{
    extern __shared__ unsigned long long pre[];      // [n_links + 1], sized at launch
    __shared__ unsigned long long list[VERIFY_LIST], list_at;
    __shared__ uint32_t n_list;
    if (threadIdx.x == 0) n_list = 0u;
    level_prefix_lds(a, pre);
    const uint32_t lane = threadIdx.x & 63u;
    const uint64_t waves = (uint64_t)gridDim.x * (VERIFY_THREADS / 64u);
    const uint64_t total = pre[a.n_links];
    // the link at hand, and the next tuple of these lanes: read while the one
    // before it is tested
    uint32_t l = ~0u, lg = 0, lanes = 0, r = 0, delta = 0, q = 0, qmask = 0, words = 0, T = 0;
    bool rehash = false;
    uint64_t n = 0, next_x = 0;
    uint32_t next_he0 = 0;
    bool next_ok = false;
    const LinkDesc* D = nullptr;
    const uint4* snap = nullptr;
    const uint64_t* in_x = nullptr;
    const uint32_t* in_h0 = nullptr;
    auto fetch = [&](uint64_t t) {
        const uint64_t idx = ((t - pre[l]) << (6u - lg)) + (lane >> lg);
        next_ok = idx < n;
        next_he0 = next_ok ? in_h0[idx] : 0u;
        next_x = next_ok ? in_x[idx] : 0ull;
    };
    for (uint64_t t = (uint64_t)(threadIdx.x >> 6) * gridDim.x + blockIdx.x; t < total; t += waves) {
        if (l == ~0u || t >= pre[l + 1]) {
            l = uniform(find_link(pre, a.n_links, t));
            D = a.links + l;
            lg = verify_lanes_log2(D->log2eta);
            lanes = 1u << lg;
            r = D->r; delta = D->delta; q = D->q; T = D->T;
            qmask = (1u << q) - 1u;
            words = D->eta >> 7;                             // 128 cells per load
            rehash = D->rehash != 0u;
            const unsigned long long raw = D->ctl->level_n[r - 3u];
            n = raw < D->max_tuples ? raw : D->max_tuples;
            // from the snapshots hot detection took of the (hot) estimators
            snap = reinterpret_cast<const uint4*>(D->live16);
            in_x = D->ctb_x[(r - 3u) & 1u];
            in_h0 = D->ctb_h0[(r - 3u) & 1u];
            fetch(t);
        }
        const uint32_t he0 = next_he0, sub = lane & (lanes - 1u);     // sub: this lane's place among its tuple's lanes
        const uint64_t x = next_x;
        bool ok = next_ok;
        if (t + waves < pre[l + 1]) fetch(t + waves);
        if (rehash && ok) ok = (tab_hash(D->tables, (uint32_t)x) & qmask) == he0;
        if (!__any(ok)) continue;
        auto row_words = [&](uint32_t i) {
            const uint32_t col = i == 0 ? he0 : (((uint32_t)(x >> ((i - 1) * delta)) & qmask) ^ he0);
            return snap + (((uint64_t)i << q) | col) * words;
        };
        // the union of rows i0 .. i1 (three at most, loaded together) with m
        auto rows_and = [&](uint4& m, uint32_t w, uint32_t i0, uint32_t i1) {
            const uint4 v0 = row_words(i0)[w], v1 = row_words(min(i0 + 1u, i1))[w], v2 = row_words(i1)[w];
            m.x &= v0.x & v1.x & v2.x; m.y &= v0.y & v1.y & v2.y;
            m.z &= v0.z & v1.z & v2.z; m.w &= v0.w & v1.w & v2.w;
        };
        // the count over all of a tuple's lanes
        auto count = [&](const uint4& m) { return (uint32_t)(__popc(m.x) + __popc(m.y) + __popc(m.z) + __popc(m.w)); };
        auto lanes_sum = [&](uint32_t v) {
            for (uint32_t o = lanes >> 1; o > 0; o >>= 1) v += __shfl_xor(v, (int)o, 64);
            return v;
        };
        uint32_t R = 0;
        for (uint32_t w0 = 0; w0 < words; w0 += lanes) {
            uint4 m = ok ? make_uint4(~0u, ~0u, ~0u, ~0u) : make_uint4(0u, 0u, 0u, 0u);
            for (uint32_t i = 0; i < r; i += 3u) {
                if (ok) rows_and(m, w0 + sub, i, min(i + 2u, r - 1u));
                // an estimator in one load per row: tuples that cannot reach T any more end here
                if (words <= 64u && i + 3u < r) {
                    ok = ok && lanes_sum(count(m)) >= T;
                    if (!__any(ok)) break;
                }
            }
            R += count(m);
        }
        R = lanes_sum(R);
        if (ok && sub == 0 && R >= T) {
            const unsigned long long key = (x << 32) | (uint64_t)(0xFFFFFFFFu - R);
            const uint32_t at = a.n_links == 1u ? atomicAdd(&n_list, 1u) : VERIFY_LIST;
            if (at < VERIFY_LIST) {
                list[at] = key;
            } else {
                const unsigned long long i = atomicAdd(&D->ctl->n_acc, 1ull);
                if (i < D->max_results) D->acc[i] = key;
            }
        }
    }
    if (a.n_links != 1u) return;
    __syncthreads();
    const uint32_t found = min(n_list, VERIFY_LIST);
    if (found == 0) return;
    if (threadIdx.x == 0) list_at = atomicAdd(&a.links->ctl->n_acc, (unsigned long long)found);
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < found; i += VERIFY_THREADS)
        if (list_at + i < a.links->max_results) a.links->acc[list_at + i] = list[i];
}

// ---------------------------------------------------------------- sort + report
// Accepted keys are (ip << 32) | (2^32-1 - R): ascending order gives ascending
// ip with the largest R first, so the first key of every ip run is kept.

__device__ __forceinline__ double estimate(uint32_t eta, uint32_t R)
{
    // Eq. 1 with z0 = eta - R, at least 1
    double z0 = (double)eta - (double)R;
    if (z0 < 1.0) z0 = 1.0;
    return -(double)eta * log(z0 / (double)eta);
}

// Links whose host mailbox is mapped (single detectors) get the control
// block written into it by the close's last kernel, instead of a copy.
__device__ __forceinline__ void ctl_to_host(const LinkDesc* D, unsigned long long n_out)
{
    if (!D->host_ctl) return;
    __syncthreads();
    const uint32_t* src = reinterpret_cast<const uint32_t*>(D->ctl);
    uint32_t* dst = reinterpret_cast<uint32_t*>(D->host_ctl);
    constexpr uint32_t words = sizeof(Ctl) / 4;
    constexpr uint32_t nout_word = offsetof(Ctl, n_out) / 4;
    if (threadIdx.x < words) {
        uint32_t v = src[threadIdx.x];
        if (threadIdx.x == nout_word) v = (uint32_t)n_out;
        if (threadIdx.x == nout_word + 1) v = (uint32_t)(n_out >> 32);
        dst[threadIdx.x] = v;
    }
}

// The list of up to sort_limit (<= SORT_SMALL) keys in two launches, ranked by
// counting: every key's ip is compared with every other, RANK_KEYS keys of a
// workgroup at a time, each by 32 lanes that share the others, read from LDS.
// n^2 comparisons spread over the chip are far cheaper than one workgroup's
// sort, a chain of log2(n)^2 / 2 barriers on one compute unit, or than a
// launch per step of it and a host that waits for the list's length (7000
// hosts: 49 us with 64 keys a workgroup, 16 lanes each, and one load in
// flight, 28 so; 11300 hosts: a close of 667 us with the multi-kernel sort,
// 350 so).
//   k_sort_keep: a key stays if no other of its ip comes before it (larger R,
//   or equal and earlier in the list); n_out counts them.  A kept key's ip
//   goes to the link's idle candidate buffers (which hold at least as many
//   tuples as passed; the flags to their he_0 half), the others become 2^32 -
//   1 there, above or equal to every ip.
//   k_sort_place: the place of a kept key is the number of kept ips below its.
// Grid: links x workgroups, each taking RANK_KEYS keys in turn.  Lists above
// the link's limit are left to the multi-kernel sort.
constexpr uint32_t RANK_KEYS = 32;
static_assert(SORT_SMALL % 128u == 0u, "ips are read in rounds of 128");

// The number of keys of this link's list that the small sort takes (0: none).
__device__ __forceinline__ uint32_t rank_keys(const LinkDesc* D)
{
    const uint64_t n = D->ctl->n_acc;
    return n > D->sort_limit || n > D->max_results ? 0u : (uint32_t)n;
}

// Idle once the tuples are tested: the kept ips, and a flag per key.
__device__ __forceinline__ uint32_t* rank_ips(const LinkDesc* D)
{
    return reinterpret_cast<uint32_t*>(D->ctb_x[((D->r - 3u) & 1u) ^ 1u]);
}
__device__ __forceinline__ uint32_t* rank_flags(const LinkDesc* D) { return D->ctb_h0[((D->r - 3u) & 1u) ^ 1u]; }

// n values of a workgroup into LDS, padded with 2^32 - 1 to whole rounds of
// 128; four loads of a thread in flight.
template <class F>
__device__ __forceinline__ void load_ips(uint32_t* ips, uint32_t n, F value)
{
    const uint32_t padded = (n + 127u) & ~127u;
    for (uint32_t i0 = threadIdx.x; i0 < padded; i0 += 4096u) {
        uint32_t v[4];
#pragma unroll
        for (uint32_t u = 0; u < 4; u++) v[u] = value(min(i0 + 1024u * u, n - 1u));
#pragma unroll
        for (uint32_t u = 0; u < 4; u++) {
            const uint32_t i = i0 + 1024u * u;
            if (i < padded) ips[i] = i < n ? v[u] : ~0u;
        }
    }
}

__global__ __launch_bounds__(1024) void k_sort_keep(const LinkDesc* links)
{
    __shared__ __align__(16) uint32_t ips[SORT_SMALL];
    __shared__ uint32_t before[RANK_KEYS];
    const LinkDesc* D = links + blockIdx.x;
    const uint32_t n = rank_keys(D), lane = threadIdx.x & (RANK_KEYS - 1u), share = threadIdx.x / RANK_KEYS;
    if (blockIdx.y * RANK_KEYS >= n) return;
    const unsigned long long* keys = D->acc;
    uint32_t *kept = rank_ips(D), *flags = rank_flags(D);
    load_ips(ips, n, [&](uint32_t i) { return (uint32_t)(keys[i] >> 32); });
    const uint4* quads = reinterpret_cast<const uint4*>(ips);
    uint32_t n_kept = 0;
    for (uint32_t i0 = blockIdx.y * RANK_KEYS; i0 < n; i0 += gridDim.y * RANK_KEYS) {
        const uint32_t i = i0 + lane;
        const unsigned long long k = i < n ? keys[i] : 0ull;
        const uint32_t ip = (uint32_t)(k >> 32);
        if (threadIdx.x < RANK_KEYS) before[lane] = 0u;
        __syncthreads();
#pragma unroll 4
        for (uint32_t j = share; 4u * j < n; j += 32u) {
            const uint4 v = quads[j];
            if (v.x != ip && v.y != ip && v.z != ip && v.w != ip) continue;
            // the key itself or, rarely, another tuple that regained its ip
            for (uint32_t o = 4u * j; o < min(n, 4u * j + 4u); o++) {
                if (ips[o] != ip || o == i) continue;
                const unsigned long long ko = keys[o];
                if (ko < k || (ko == k && o < i)) before[lane] = 1u;
            }
        }
        __syncthreads();
        if (threadIdx.x < RANK_KEYS && i < n) {
            const bool stays = !before[lane];
            kept[i] = stays ? ip : ~0u;
            flags[i] = stays ? 1u : 0u;
            n_kept += (uint32_t)__popcll(__ballot(stays));
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) atomicAdd(&D->ctl->n_out, (unsigned long long)n_kept);
}

// next: the hot bitmasks, read for the last time by the expansion, are cleared
// and the next slot's constants formed from this one's, so that its close
// starts with the detection (a launch of k_prepare before it cost a slot 2 to 3
// us).
__global__ __launch_bounds__(1024) void k_sort_place(LinkDesc* links, uint32_t next)
{
    __shared__ __align__(16) uint32_t ips[SORT_SMALL];
    __shared__ uint32_t below[RANK_KEYS];
    const LinkDesc* D = links + blockIdx.x;
    const uint32_t n = rank_keys(D), lane = threadIdx.x & (RANK_KEYS - 1u), share = threadIdx.x / RANK_KEYS;
    const uint32_t *kept = rank_ips(D), *flags = rank_flags(D);
    if (blockIdx.y * RANK_KEYS < n) load_ips(ips, n, [&](uint32_t i) { return kept[i]; });
    const uint4* quads = reinterpret_cast<const uint4*>(ips);
    for (uint32_t i0 = blockIdx.y * RANK_KEYS; i0 < n; i0 += gridDim.y * RANK_KEYS) {
        const uint32_t i = i0 + lane;
        const bool stays = i < n && flags[i];
        if (threadIdx.x < RANK_KEYS) below[lane] = 0u;
        __syncthreads();
        const uint32_t ip = i < n ? ips[i] : 0u;
        uint32_t c = 0;
#pragma unroll 4
        for (uint32_t j = share; 4u * j < n; j += 32u) {
            const uint4 v = quads[j];
            c += (v.x < ip ? 1u : 0u) + (v.y < ip ? 1u : 0u) + (v.z < ip ? 1u : 0u) + (v.w < ip ? 1u : 0u);
        }
        if (c) atomicAdd(&below[lane], c);
        __syncthreads();
        if (threadIdx.x < RANK_KEYS && stays) {
            const uint32_t at = below[lane], R = 0xFFFFFFFFu - (uint32_t)D->acc[i];
            SuperPointDev sp;
            sp.ip = ip; sp.rk = R; sp.est = estimate(D->eta, R);
            if (at < D->host_cap) D->host_out[at] = sp;       // straight into the host's pinned mailbox
            D->out[at] = sp;
        }
        __syncthreads();
    }
    if (next) {
        uint32_t* p = reinterpret_cast<uint32_t*>(D->hotbits);     // hotT follows hotbits
        for (uint64_t i = blockIdx.y * 1024u + threadIdx.x; i < D->hot_words; i += gridDim.y * 1024u) p[i] = 0u;
        if (blockIdx.y == gridDim.y - 1u && threadIdx.x == 0) {
            LinkDesc* N = links + blockIdx.x;
            const bool cell16 = D->cell16 != 0u;
            const uint32_t cur = D->cur == (cell16 ? 65535u : 255u) ? 1u : D->cur + 1u;
            const uint32_t phase = D->expire_phase + 1u;
            N->L = live_cfg(cur, D->k, cell16);
            N->cur = cur;
            N->expire_phase = phase == D->expire_period ? 0u : phase;
        }
    }
    if (blockIdx.y != 0) return;
    // the link's first workgroup ends its close: the next slot opens (a list
    // left to the multi-kernel sort is finished by the host)
    ctl_to_host(D, D->ctl->n_out);
    if (threadIdx.x == 0) D->clock->t += 1ull;
}

// Global bitonic step over N (power of two) keys, for lists above SORT_SMALL.
__global__ __launch_bounds__(256) void k_bitonic_step(unsigned long long* keys, uint64_t N, uint64_t j, uint64_t k)
{
    const uint64_t stride = (uint64_t)gridDim.x * 256u;
    for (uint64_t i = (uint64_t)blockIdx.x * 256u + threadIdx.x; i < N; i += stride) {
        const uint64_t p = i ^ j;
        if (p > i) {
            const unsigned long long u = keys[i], v = keys[p];
            const bool up = (i & k) == 0;
            if ((u > v) == up) { keys[i] = v; keys[p] = u; }
        }
    }
}

// Pad keys[n..N) with the largest key.
__global__ void k_pad_keys(unsigned long long* dst, const unsigned long long* src, uint64_t n, uint64_t N)
{
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < N; i += stride)
        dst[i] = i < n ? src[i] : ~0ull;
}

// Single block: de-duplicate n sorted keys into the link's result list.
__global__ __launch_bounds__(1024) void k_dedup_sorted(const LinkDesc* D, const unsigned long long* sorted, uint64_t n)
{
    __shared__ uint32_t lds[16];
    uint64_t out_base = 0;
    const uint32_t CHUNK = 8192u;
    for (uint64_t c0 = 0; c0 < n; c0 += CHUNK) {
        const uint64_t c1 = c0 + CHUNK < n ? c0 + CHUNK : n;
        const uint64_t i0 = c0 + (uint64_t)threadIdx.x * 8u;
        const uint64_t i1 = i0 + 8u < c1 ? i0 + 8u : c1;
        uint32_t cnt = 0;
        for (uint64_t i = i0; i < i1; i++) cnt += (i == 0 || (sorted[i] >> 32) != (sorted[i - 1] >> 32));
        uint32_t total;
        uint32_t off = block_exclusive_scan_1024(cnt, lds, &total);
        uint64_t o = out_base + off;
        for (uint64_t i = i0; i < i1; i++) {
            if (i == 0 || (sorted[i] >> 32) != (sorted[i - 1] >> 32)) {
                const uint32_t R = 0xFFFFFFFFu - (uint32_t)sorted[i];
                SuperPointDev sp;
                sp.ip = (uint32_t)(sorted[i] >> 32); sp.rk = R; sp.est = estimate(D->eta, R);
                D->out[o++] = sp;
            }
        }
        out_base += total;
    }
    if (threadIdx.x == 0) D->ctl->n_out = out_base;
}

// One block per link: copy the link's list behind those of the links before it
// into one packed array (up to cap entries in total) and record the offsets.
__global__ __launch_bounds__(256) void k_pack(PackArgs a)
{
    const uint32_t l = blockIdx.x;
    unsigned long long off = 0;
    for (uint32_t j = 0; j < l; j++) off += a.links[j].ctl->n_out;
    const LinkDesc* D = a.links + l;
    const unsigned long long n = D->ctl->n_out;
    if (threadIdx.x == 0) {
        a.offsets[l] = off;
        if (l == a.n_links - 1) a.offsets[a.n_links] = off + n;
    }
    for (unsigned long long i = threadIdx.x; i < n; i += 256u)
        if (off + i < a.cap) a.packed[off + i] = D->out[i];
}

// ---------------------------------------------------------------- merge
// Alg. 5 with the per-cell most recent hit over the routers: for every cell the
// stamp with the smallest distance wins; cells not live anywhere become empty.
//
// Distances are compared as x = (cur - stamp) mod 256, two cells to a 32-bit
// word: the distance for stamps up to cur, one more than it for the others
// (stamps run modulo 255), so their order is the distances'; an empty cell (x
// = cur, between the two) gets a bit above all of them.  The winner's stamp is
// cur - x again.  HBM bound: a workgroup streams 16 KiB of every source in
// turn, so that the sources' pages are not opened by turns chunk by chunk, and
// a word of four cells takes about 16 vector instructions a source (byte by
// byte 50, as long as the loads).  Measured on 16 states of 320 MiB, 5.7 GB
// read and written: 1131 us a chunk of each source at a time, byte by byte;
// 1080 in 16 KiB pieces; 963 (5.9 TB/s) with non-temporal loads.
constexpr uint32_t MERGE_CHUNKS = 4;

__device__ __forceinline__ uint32_t pk_min_u16(uint32_t a, uint32_t b)
{
    typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(u16x2, a), __builtin_bit_cast(u16x2, b)));
}

__device__ __forceinline__ uint32_t pk_sub_u16(uint32_t a, uint32_t b)
{
    typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_bit_cast(u16x2, a) - __builtin_bit_cast(u16x2, b));
}

// x of the cells in the low bytes of e's halves, above 255 for empty ones
__device__ __forceinline__ uint32_t merge_age(uint32_t e, uint32_t cur2)
{
    const uint32_t M = 0x00FF00FFu, H = 0x01000100u;
    return (pk_sub_u16(cur2, e) & M) | (~(e + M) & H);
}

__global__ __launch_bounds__(256) void k_merge(MergeArgs a)
{
    const uint32_t M = 0x00FF00FFu;
    const uint32_t cur2 = a.cur * 0x00010001u;
    // live: x < k for stamps up to cur, x - 1 < k for the older ones past the wrap
    const uint32_t kx = a.k > a.cur ? a.k + 1u : a.k;
    const uint64_t stride = (uint64_t)gridDim.x * 256u * MERGE_CHUNKS;
    for (uint64_t i0 = (uint64_t)blockIdx.x * 256u * MERGE_CHUNKS + threadIdx.x; i0 < a.n16; i0 += stride) {
        uint32_t even[MERGE_CHUNKS][4], odd[MERGE_CHUNKS][4];
#pragma unroll
        for (uint32_t c = 0; c < MERGE_CHUNKS; c++)
#pragma unroll
            for (int w = 0; w < 4; w++) even[c][w] = odd[c][w] = 0x01FF01FFu;
#pragma unroll 1
        for (uint32_t j = 0; j < a.n_src; j++) {
            const uint4* src = reinterpret_cast<const uint4*>(a.src[j]);
            uint4 v[MERGE_CHUNKS];
#pragma unroll
            for (uint32_t c = 0; c < MERGE_CHUNKS; c++) v[c] = load_stream(src + (i0 + 256u * c < a.n16 ? i0 + 256u * c : i0));
#pragma unroll
            for (uint32_t c = 0; c < MERGE_CHUNKS; c++) {
                const uint32_t x[4] = {v[c].x, v[c].y, v[c].z, v[c].w};
#pragma unroll
                for (int w = 0; w < 4; w++) {
                    even[c][w] = pk_min_u16(even[c][w], merge_age(x[w] & M, cur2));
                    odd[c][w] = pk_min_u16(odd[c][w], merge_age((x[w] >> 8) & M, cur2));
                }
            }
        }
#pragma unroll
        for (uint32_t c = 0; c < MERGE_CHUNKS; c++) {
            uint32_t o[4];
#pragma unroll
            for (int w = 0; w < 4; w++) {
                auto stamps = [&](uint32_t x) {
                    const uint32_t s = pk_sub_u16(cur2, x) & M;
                    return ((x & 0xFFFFu) < kx ? s & 0xFFFFu : 0u) | ((x >> 16) < kx ? s & 0xFFFF0000u : 0u);
                };
                o[w] = stamps(even[c][w]) | stamps(odd[c][w]) << 8;
            }
            if (i0 + 256u * c < a.n16) reinterpret_cast<uint4*>(a.dst)[i0 + 256u * c] = make_uint4(o[0], o[1], o[2], o[3]);
        }
    }
}

// The same for 16-bit cells: eight per chunk, distances modulo 65535.
__global__ __launch_bounds__(256) void k_merge16(MergeArgs a)
{
    const uint64_t stride = (uint64_t)gridDim.x * 256u;
    for (uint64_t i = (uint64_t)blockIdx.x * 256u + threadIdx.x; i < a.n16; i += stride) {
        uint32_t best[8];
        uint32_t code[8];
#pragma unroll
        for (int b = 0; b < 8; b++) { best[b] = 65535u; code[b] = 0u; }
        for (uint32_t j = 0; j < a.n_src; j++) {
            const uint4 v = reinterpret_cast<const uint4*>(a.src[j])[i];
            if ((v.x | v.y | v.z | v.w) == 0u) continue;
            const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int b = 0; b < 8; b++) {
                const uint32_t c = (w[b >> 1] >> ((b & 1) * 16)) & 0xFFFFu;
                if (c) {
                    int age = (int)a.cur - (int)c;
                    if (age < 0) age += 65535;
                    if ((uint32_t)age < best[b]) { best[b] = (uint32_t)age; code[b] = c; }
                }
            }
        }
        uint32_t o[4] = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int b = 0; b < 8; b++)
            if (best[b] < a.k) o[b >> 1] |= code[b] << ((b & 1) * 16);
        reinterpret_cast<uint4*>(a.dst)[i] = make_uint4(o[0], o[1], o[2], o[3]);
    }
}

// ---------------------------------------------------------------- canonical

// Distance of every cell (t - slot of its latest hit) where it is below k,
// else 0xFFFF; stamps modulo M = 255 (8-bit cells) or 65535 (16-bit).
template <class T, int M>
__global__ __launch_bounds__(256) void k_canonical(const uint8_t* state, uint16_t* out, uint64_t n, uint32_t cur, uint32_t k)
{
    const uint64_t stride = (uint64_t)gridDim.x * 256u;
    const T* cells = reinterpret_cast<const T*>(state);
    for (uint64_t i = (uint64_t)blockIdx.x * 256u + threadIdx.x; i < n; i += stride) {
        const uint32_t c = cells[i];
        uint32_t v = 0xFFFFu;
        if (c) {
            int age = (int)cur - (int)c;
            if (age < 0) age += M;
            if ((uint32_t)age < k) v = (uint32_t)age;
        }
        out[i] = (uint16_t)v;
    }
}

// ---------------------------------------------------------------- launchers

static dim3 grid_for(uint64_t n, uint32_t block, uint32_t max_blocks)
{
    uint64_t g = (n + block - 1) / block;
    if (g < 1) g = 1;
    if (g > max_blocks) g = max_blocks;
    return dim3((uint32_t)g);
}

hipError_t launch_fill_u32(uint32_t* p, uint64_t n, uint32_t v, hipStream_t s)
{
    k_fill_u32<<<grid_for(n, 256, 8192), 256, 0, s>>>(p, n, v);
    return hipGetLastError();
}

hipError_t launch_prepare(const LinkDesc* links, uint32_t n_links, hipStream_t s)
{
    k_prepare<<<dim3(n_links, 16), 256, 0, s>>>(const_cast<LinkDesc*>(links));
    return hipGetLastError();
}

hipError_t launch_expire(const ExpireArgs& a, bool cell16, hipStream_t s)
{
    if (a.period == 0 || a.chunks < 64u) return hipErrorInvalidValue;
    const uint32_t waves = (uint32_t)((a.n_se + a.period - 1) / a.period), grid = (waves + 3u) / 4u;
    if (cell16) k_expire<true><<<grid, 256, 0, s>>>(a);
    else k_expire<false><<<grid, 256, 0, s>>>(a);
    return hipGetLastError();
}

hipError_t launch_gather_ctl(const LinkDesc* links, uint32_t n_links, Ctl* dst, hipStream_t s)
{
    k_gather_ctl<<<grid_for(n_links, 256, 64), 256, 0, s>>>(links, n_links, dst);
    return hipGetLastError();
}



hipError_t launch_scan(const ScanArgs& a, hipStream_t s)
{
    // by eighths: as many workgroups for every eighth of the window
    const dim3 g = a.eighths ? dim3(8u * grid_for(a.n, 256, 256).x) : grid_for(a.n, 256, 256 * 16);
    if (a.cell16) k_scan<uint16_t><<<g, 256, 0, s>>>(a);
    else k_scan<uint8_t><<<g, 256, 0, s>>>(a);
    return hipGetLastError();
}

hipError_t launch_scan_counted(const LinkDesc* link, const uint2* pairs, uint64_t n, uint32_t stamp, uint32_t slot, hipStream_t s)
{
    k_scan_counted<<<grid_for(n, 256, 2048), 256, 0, s>>>(link, pairs, n, stamp, slot);
    return hipGetLastError();
}

hipError_t launch_scan_tiles(const TileScanArgs& a, uint32_t blocks, hipStream_t s)
{
    k_scan_tiles<<<blocks, 256, 0, s>>>(a);
    return hipGetLastError();
}

// Kernels of more dynamic LDS than the default (kernel, bytes) are set up once
// on every device, whichever thread launches one of them first.
static hipError_t set_lds(std::atomic<uint64_t>& done, std::initializer_list<std::pair<const void*, uint64_t>> kernels)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t bit = dev < 64 ? 1ull << dev : 0ull;
    if (done.load(std::memory_order_acquire) & bit) return hipSuccess;
    for (const auto& k : kernels) {
        e = hipFuncSetAttribute(k.first, hipFuncAttributeMaxDynamicSharedMemorySize, (int)k.second);
        if (e != hipSuccess) return e;
    }
    done.fetch_or(bit, std::memory_order_release);
    return hipSuccess;
}

static hipError_t bin_lds_attr()
{
    static std::atomic<uint64_t> done{0};
    return set_lds(done, {{reinterpret_cast<const void*>(&k_bin<0, 0, false>), BIN_LDS_WORDS * 4u},
                          {reinterpret_cast<const void*>(&k_bin<6, 6, false>), BIN_LDS_WORDS * 4u},
                          {reinterpret_cast<const void*>(&k_bin<5, 7, false>), BIN_LDS_WORDS * 4u},
                          {reinterpret_cast<const void*>(&k_bin_multi_rows<false>), BIN_LDS_WORDS * 4u},
                          {reinterpret_cast<const void*>(&k_bin<0, 0, true>), BIN_HALF_WORDS * 4u},
                          {reinterpret_cast<const void*>(&k_bin<6, 3, true>), BIN_HALF_WORDS * 4u},
                          {reinterpret_cast<const void*>(&k_bin<5, 4, true>), BIN_HALF_WORDS * 4u},
                          {reinterpret_cast<const void*>(&k_bin_multi_rows<true>), BIN_HALF_WORDS * 4u}});
}

bool bin_half(const BinArgs& a) { return bin_lds_words(a.n_bins, a.pb, a.r) <= BIN_HALF_WORDS; }

uint32_t bin_workgroups(const BinArgs& a)      // segments dealt to XCDs in eighths
{
    return 8u * (((a.blocks + 7u) / 8u + a.rounds - 1u) / a.rounds);
}

hipError_t launch_bin(const BinArgs& a, hipStream_t s)
{
    const uint32_t words = bin_lds_words(a.n_bins, a.pb, a.r);
    if (a.blocks == 0 || a.rounds == 0 || words > BIN_LDS_WORDS || !bin_items_aligned(a)) return hipErrorInvalidValue;
    hipError_t e = bin_lds_attr();
    if (e != hipSuccess) return e;
    const uint32_t grid = bin_workgroups(a), lds = words * 4u;
    if (bin_half(a)) {
        if (a.r == 6 && a.pb <= 3u * 1024u) k_bin<6, 3, true><<<grid, 1024, lds, s>>>(a);
        else if (a.r == 5 && a.pb <= 4u * 1024u) k_bin<5, 4, true><<<grid, 1024, lds, s>>>(a);
        else k_bin<0, 0, true><<<grid, 1024, lds, s>>>(a);
    } else {
        if (a.r == 6 && a.pb <= 6u * 1024u) k_bin<6, 6, false><<<grid, 1024, lds, s>>>(a);
        else if (a.r == 5 && a.pb <= 7u * 1024u) k_bin<5, 7, false><<<grid, 1024, lds, s>>>(a);
        else k_bin<0, 0, false><<<grid, 1024, lds, s>>>(a);
    }
    return hipGetLastError();
}

hipError_t launch_bin_multi(const MultiBinArgs& m, uint32_t total_wg, bool half, hipStream_t s)
{
    if (m.n == 0 || total_wg == 0) return hipErrorInvalidValue;
    hipError_t e = bin_lds_attr();
    if (e != hipSuccess) return e;
    // every link's plan fits the LDS
    if (half) k_bin_multi_rows<true><<<total_wg, 1024, BIN_HALF_WORDS * 4u, s>>>(m);
    else k_bin_multi_rows<false><<<total_wg, 1024, BIN_LDS_WORDS * 4u, s>>>(m);
    return hipGetLastError();
}

uint32_t apply_workgroups(const ApplyArgs& a) { return (uint32_t)(8ull * a.parts * ((a.n_bins + 7u) / 8u)); }
uint32_t apply_counted_workgroups(const ApplyArgs& a) { return 8u * ((a.n_bins + 7u) / 8u); }

hipError_t launch_apply_multi(const MultiApplyArgs& m, uint32_t total_wg, hipStream_t s)
{
    if (m.n == 0 || total_wg == 0) return hipErrorInvalidValue;
    k_apply_multi<true><<<total_wg, 64, 0, s>>>(m);
    return hipGetLastError();
}

hipError_t launch_apply(const ApplyArgs& a, hipStream_t s)
{
    if (a.parts == 0 || a.per_part == 0) return hipErrorInvalidValue;
    const uint32_t grid = apply_workgroups(a);
    if (a.cell16) {
        if (a.pack) k_apply<true, uint16_t><<<grid, 64, 0, s>>>(a);
        else k_apply<false, uint16_t><<<grid, 64, 0, s>>>(a);
    } else {
        if (a.pack) k_apply<true, uint8_t><<<grid, 64, 0, s>>>(a);
        else k_apply<false, uint8_t><<<grid, 64, 0, s>>>(a);
    }
    return hipGetLastError();
}

hipError_t launch_apply_marked16(const ApplyArgs& a, hipStream_t s)
{
    if (!a.cell16 || !a.pack || a.bin_shift < 10 || a.bin_shift > MARKED16_MAX_SHIFT) return hipErrorInvalidValue;
    const uint32_t lds = (1u << (a.bin_shift - 5u)) * 4u;      // the bitmap
    static std::atomic<uint64_t> done{0};
    hipError_t e = set_lds(done, {{reinterpret_cast<const void*>(&k_apply_marked16), MARKED16_LDS_MAX}});
    if (e != hipSuccess) return e;
    k_apply_marked16<<<apply_counted_workgroups(a), 64 * CAPPLY_WAVES, lds, s>>>(a);
    return hipGetLastError();
}

static hipError_t counted_lds_attr()
{
    static std::atomic<uint64_t> done{0};
    return set_lds(done, {{reinterpret_cast<const void*>(&k_apply_counted), COUNTED_LDS_BYTES},
                          {reinterpret_cast<const void*>(&k_apply_counted_multi), COUNTED_LDS_BYTES}});
}

hipError_t launch_apply_counted(const ApplyArgs& a, hipStream_t s)
{
    const uint64_t bytes = counted_lds_bytes(a.bin_shift, a.log2eta, a.k);
    if (!a.counts || a.k == 0 || a.slot >= a.k || a.bin_shift < a.log2eta || a.bin_shift < 5 ||
        bytes > COUNTED_LDS_BYTES || a.n_bins == 0)
        return hipErrorInvalidValue;
    // counted bins are at most 2 MiB: always packed, and a segment of one offset
    // or more is at least the pair of words that mark_runs reads at a time
    if (!a.pack || a.seg == 0) return hipErrorInvalidValue;
    if (a.cell16) return hipErrorInvalidValue;                   // counters are kept for 8-bit cells only
    hipError_t e = counted_lds_attr();
    if (e != hipSuccess) return e;
    k_apply_counted<<<apply_counted_workgroups(a), 64 * CAPPLY_WAVES, (uint32_t)bytes, s>>>(a);
    return hipGetLastError();
}

hipError_t launch_apply_counted_multi(const MultiApplyArgs& m, uint32_t total_wg, uint32_t lds_bytes, hipStream_t s)
{
    if (m.n == 0 || total_wg == 0 || lds_bytes > COUNTED_LDS_BYTES) return hipErrorInvalidValue;
    hipError_t e = counted_lds_attr();
    if (e != hipSuccess) return e;
    k_apply_counted_multi<<<total_wg, 64 * CAPPLY_WAVES, lds_bytes, s>>>(m);
    return hipGetLastError();
}

hipError_t launch_count(const LinkDesc* link, uint64_t n_se, hipStream_t s)
{
    if (n_se == 0) return hipErrorInvalidValue;
    k_count<<<(uint32_t)((n_se + 255u) / 256u), 256, 0, s>>>(link, n_se);
    return hipGetLastError();
}

uint32_t count_workgroups(uint64_t n_se) { return (uint32_t)((n_se + 255u) / 256u); }

hipError_t launch_count_multi(const CountMultiArgs& m, uint32_t total_wg, hipStream_t s)
{
    if (m.n == 0 || total_wg == 0) return hipErrorInvalidValue;
    k_count_multi<<<total_wg, 256, 0, s>>>(m);
    return hipGetLastError();
}

hipError_t launch_recount(const LinkDesc* link, uint64_t n_se, hipStream_t s)
{
    if (n_se == 0) return hipErrorInvalidValue;
    k_recount<<<(uint32_t)((n_se + 3u) / 4u), 256, 0, s>>>(link, n_se);
    return hipGetLastError();
}

template <int CH, bool SMALL>
static void hot_detect(const DetectArgs& a, hipStream_t s)
{
    const dim3 g((uint32_t)((a.total + DETECT_WAVES - 1) / DETECT_WAVES));
    if (a.stream) k_hot_detect<CH, SMALL, true><<<g, 64u * DETECT_WAVES, 0, s>>>(a);
    else k_hot_detect<CH, SMALL, false><<<g, 64u * DETECT_WAVES, 0, s>>>(a);
}

hipError_t launch_hot_detect(const DetectArgs& a, uint32_t max_chunks_per_lane, bool small, hipStream_t s)
{
    // SMALL: some link has eta < 4096 (several estimators per wave) or the
    // engine has several links (link prefix in LDS); the plain variant keeps
    // half the registers, so more waves stream the state
    if (small) {
        if (max_chunks_per_lane >= 8) hot_detect<8, true>(a, s);
        else hot_detect<4, true>(a, s);
    } else {
        if (max_chunks_per_lane >= 8) hot_detect<8, false>(a, s);
        else hot_detect<4, false>(a, s);        // eta = 4096
    }
    return hipGetLastError();
}

hipError_t launch_hot_detect16(const DetectArgs& a, hipStream_t s)
{
    if (a.n_links != 1 || a.total == 0) return hipErrorInvalidValue;
    const dim3 g((uint32_t)((a.total + DETECT_WAVES - 1) / DETECT_WAVES));
    if (a.stream) k_hot_detect16<4, true><<<g, 64u * DETECT_WAVES, 0, s>>>(a);
    else k_hot_detect16<4, false><<<g, 64u * DETECT_WAVES, 0, s>>>(a);
    return hipGetLastError();
}

hipError_t launch_hot_compact(const LinkDesc* links, const uint32_t* row_table, uint32_t rows, hipStream_t s)
{
    k_hot_compact<<<rows, 1024, 0, s>>>(links, row_table);
    return hipGetLastError();
}


// dynamic LDS of the level kernels: the work prefix over the links
static inline size_t prefix_lds(const LevelArgs& a) { return ((size_t)a.n_links + 1) * 8u; }

hipError_t launch_expand0(const LevelArgs& a, hipStream_t s)
{
    k_expand0<<<2048, 256, prefix_lds(a), s>>>(a);
    return hipGetLastError();
}

// workgroups of the depth-first expansion: one per compute unit (its LDS); of
// the nested walk: each flushes its counts with one atomic per level, so
// fewer is better until the grid stops filling the chip
constexpr uint32_t DFS_BLOCKS = 256, NESTED_BLOCKS = 512;
constexpr uint32_t VERIFY_BLOCKS = 512;         // two workgroups of 16 waves per compute unit

// dynamic LDS of k_expand_dfs
static uint64_t dfs_lds_bytes(uint32_t n_links, uint32_t rows, uint32_t waves, uint64_t table_bytes)
{
    return ((n_links + 2u) & ~1u) * 8ull + (uint64_t)waves * (rows * DFS_QUEUE * 16u + DFS_OUT * 8u) +
           2ull * DFS_LIST * 4u + table_bytes;
}

hipError_t launch_expand_dfs(LevelArgs a, uint32_t max_r, uint32_t max_delta, uint64_t table_bytes, hipStream_t s)
{
    if (max_r < 3 || max_r > 8) return hipErrorInvalidValue;
    // eight waves' queues at r <= 6 (64 KiB at six rows), four at r <= 8 (48 KiB at eight)
    const uint32_t waves = max_r <= 6 ? 8u : 4u;
    const uint64_t lds = dfs_lds_bytes(a.n_links, max_r - 2u, waves, table_bytes);
    if (lds > DFS_LDS_BYTES || max_delta > 6) {
        a.level = 0;
        if (max_r <= 6) k_expand_nested<6><<<NESTED_BLOCKS, 256, prefix_lds(a), s>>>(a);
        else k_expand_nested<8><<<NESTED_BLOCKS, 256, prefix_lds(a), s>>>(a);
        return hipGetLastError();
    }
    a.level = LEVEL_DFS;
    a.queue_rows = max_r - 2u;
    static std::atomic<uint64_t> done{0};
    hipError_t e = set_lds(done, {{reinterpret_cast<const void*>(&k_expand_dfs<4, 8>), DFS_LDS_BYTES},
                                  {reinterpret_cast<const void*>(&k_expand_dfs<6, 4>), DFS_LDS_BYTES}});
    if (e != hipSuccess) return e;
    if (max_r <= 6) k_expand_dfs<4, 8><<<DFS_BLOCKS, 512, (uint32_t)lds, s>>>(a);
    else k_expand_dfs<6, 4><<<DFS_BLOCKS, 256, (uint32_t)lds, s>>>(a);
    return hipGetLastError();
}

hipError_t launch_extend(const LevelArgs& a, hipStream_t s)
{
    k_extend<<<2048, 256, prefix_lds(a), s>>>(a);
    return hipGetLastError();
}

hipError_t launch_verify(const LevelArgs& a, hipStream_t s)
{
    k_verify<<<VERIFY_BLOCKS, VERIFY_THREADS, prefix_lds(a), s>>>(a);
    return hipGetLastError();
}

hipError_t launch_sort_small(LinkDesc* links, uint32_t n_links, bool next, hipStream_t s)
{
    // one link: a workgroup for every compute unit; several links share the chip
    const dim3 g(n_links, n_links == 1 ? 256u : 16u);
    k_sort_keep<<<g, 1024, 0, s>>>(links);
    k_sort_place<<<g, 1024, 0, s>>>(links, next ? 1u : 0u);
    return hipGetLastError();
}

hipError_t launch_sort_large(const LinkDesc* link, const LinkDesc& host_copy, unsigned long long* tmp, uint64_t n,
                             hipStream_t s)
{
    uint64_t N = 1;
    while (N < n) N <<= 1;
    k_pad_keys<<<grid_for(N, 256, 8192), 256, 0, s>>>(tmp, host_copy.acc, n, N);
    for (uint64_t k = 2; k <= N; k <<= 1)
        for (uint64_t j = k >> 1; j > 0; j >>= 1)
            k_bitonic_step<<<grid_for(N, 256, 8192), 256, 0, s>>>(tmp, N, j, k);
    k_dedup_sorted<<<1, 1024, 0, s>>>(link, tmp, n);
    return hipGetLastError();
}

hipError_t launch_pack(const PackArgs& a, hipStream_t s)
{
    k_pack<<<a.n_links, 256, 0, s>>>(a);
    return hipGetLastError();
}

hipError_t launch_merge(const MergeArgs& a, hipStream_t s)
{
    if (a.cell16) k_merge16<<<grid_for(a.n16, 256, 256 * 16), 256, 0, s>>>(a);
    else k_merge<<<grid_for(a.n16, 256 * MERGE_CHUNKS, 1u << 20), 256, 0, s>>>(a);
    return hipGetLastError();
}

hipError_t launch_canonical(const uint8_t* state, uint16_t* out, uint64_t n, uint32_t cur, uint32_t k, bool cell16,
                            hipStream_t s)
{
    if (cell16) k_canonical<uint16_t, 65535><<<grid_for(n, 256, 256 * 16), 256, 0, s>>>(state, out, n, cur, k);
    else k_canonical<uint8_t, 255><<<grid_for(n, 256, 256 * 16), 256, 0, s>>>(state, out, n, cur, k);
    return hipGetLastError();
}

}  // namespace ssd
