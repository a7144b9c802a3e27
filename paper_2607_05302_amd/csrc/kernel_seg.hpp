// Sorting many arrays at once, or one, out of place between the caller's planes and a
// scratch area (the paper hands arrays smaller than T to an out-of-place sort, Sec. 5):
// the LSD sort of Alg. 1 on 8-bit digits over tiles of all the arrays of a group, whose
// records together fit the scratch.  The caller's workspace holds the scratch, so a batch
// far larger than it is sorted group by group, and a group's records stay in the GPU's
// last-level cache from one round to the next.
//
// Per group: one pass counts the digits of every key position of every array
// (k_seg_hist; the last workgroup of an array turns the counts into element starts and
// finds the rounds whose digit varies), then one launch per round (k_seg_round).  A tile
// finds its digit starts by a decoupled look-back over the earlier tiles of its own array
// only; many arrays are in flight at once, so the chain of one does not set the pace.  An
// array runs an even number of rounds, so that it ends where it began: the rounds of
// constant digits are left out, but one of them if the others are odd in number.
//
// What bounds it: like the Radsort round, the latency of a tile's steps against the tiles in
// flight (two workgroups of the larger shapes per compute unit).  4096 arrays of 2^10 .. 2^22
// uint32 pairs: 137.4 ms with one workgroup per array, 44.8 ms here; one array of 49 275
// pairs 192 us by Radsort, 41 us here; the out-of-place sort of 10^7 pairs 358 us with
// k_round, 260 us here (the last two with the copy of the input).
#pragma once

#include "common.hpp"
#include "kernel_tile.hpp"

namespace rs {

struct SegArr {
    uint64_t o0;      // first element in the caller's planes
    uint32_t n;       // elements
    uint32_t scr64;   // first record in the scratch planes, in units of 64
    uint32_t tile0;   // the array's first tile
    uint32_t group;
};

// Look-back word of (tile, digit): the tile's count, or the count of its array up to and
// including the tile, and the round it belongs to, so that a group's words are cleared once.
constexpr uint32_t kSegAgg = 1u << 30, kSegIncl = 2u << 30, kSegStatus = 3u << 30;
constexpr uint32_t kSegValueBits = 26;
constexpr uint32_t kSegValue = (1u << kSegValueBits) - 1;
__device__ __forceinline__ uint32_t seg_tag(uint32_t r) { return (r + 1) << kSegValueBits; }
constexpr uint32_t kSegTag = 15u << kSegValueBits;

template <int KB, int VB> struct SegArgs {
    using K = typename UInt<KB>::T;
    using V = typename Payload<VB>::T;
    K* Ak;                 // the caller's planes
    V* Av;
    K* Sk;                 // scratch planes
    V* Sv;
    const SegArr* arr;     // all arrays of the path
    uint32_t* map;         // tile -> array
    uint32_t a0, t0;       // first array and first tile of the group
    uint32_t* hist;        // [array of the group][n_t][256]: counts, then element starts
    uint32_t* arrived;     // [array of the group]: tiles counted
    uint32_t* rounds;      // [array of the group]: bit r: round r runs; 0 until counted
    uint32_t* state;       // [tile of the group][256]: look-back words
    uint32_t* ctr;         // [n_t]: tiles claimed
    uint32_t* err;
    uint32_t r;            // round
    uint32_t na, group;    // arrays of the group, its number (k_seg_hist)
};

// The arrays of lo < n <= hi elements in order, with their scratch places and tiles: the
// running sum of their sizes in units of 64 records is cut into groups of G64.  One workgroup.
// The host laid the tables out and chose the launches by its copy of the offsets.  Where the
// device's give another number of arrays or tiles, every entry is marked unused, and the
// counting pass reports the first tile it looks at.
template <int NT>
__global__ __launch_bounds__(NT) void k_seg_plan(const uint64_t* __restrict__ offsets,
                                                 uint32_t nseg, uint64_t lo, uint64_t hi,
                                                 uint32_t G64, uint32_t E, SegArr* arr,
                                                 uint32_t count, uint32_t* map, uint32_t tiles)
{
    __shared__ uint32_t a[NT], b[NT], c[NT], tmp[NT / 64 + 1];
    uint32_t idx = 0, pos = 0, tile = 0;
    for (uint32_t i0 = 0; i0 < nseg; i0 += NT) {
        const uint32_t i = i0 + threadIdx.x;
        uint64_t o0 = 0, n = 0;
        if (i < nseg) {
            o0 = offsets[i];
            const uint64_t o1 = offsets[i + 1];
            n = o1 > o0 ? o1 - o0 : 0;
            if (n <= lo || n > hi) n = 0;
        }
        a[threadIdx.x] = n != 0;
        b[threadIdx.x] = (uint32_t)((n + 63) / 64);
        c[threadIdx.x] = (uint32_t)((n + E - 1) / E);
        __syncthreads();
        const uint32_t na = block_excl_scan<NT>(a, NT, tmp);
        const uint32_t nb = block_excl_scan<NT>(b, NT, tmp);
        const uint32_t nc = block_excl_scan<NT>(c, NT, tmp);
        const uint32_t at = idx + a[threadIdx.x], p = pos + b[threadIdx.x];
        if (n && at < count)
            arr[at] = SegArr{o0, (uint32_t)n, p % G64, tile + c[threadIdx.x], p / G64};
        idx += na;
        pos += nb;
        tile += nc;
        __syncthreads();
    }
    if (idx == count && tile == tiles) return;
    wg_global_handoff();  // the entries above land before the marks
    for (uint32_t i = threadIdx.x; i < count; i += NT) arr[i] = SegArr{0, 0, 0, 0, 0};
    for (uint32_t t = threadIdx.x; t < tiles; t += NT) map[t] = ~0u;
}

// map[tile] = array
__global__ void k_seg_map(const SegArr* __restrict__ arr, uint32_t E, uint32_t tiles,
                          uint32_t* __restrict__ map)
{
    const SegArr a = arr[blockIdx.x];
    const uint32_t nt = (a.n + E - 1) / E;
    for (uint32_t t = threadIdx.x; t < nt; t += blockDim.x)
        if (a.tile0 + t < tiles) map[a.tile0 + t] = blockIdx.x;
}

// Clears `words` words and, for a lone array, writes its entry (its map is all zeros).
__global__ void k_seg_clear(uint32_t* __restrict__ p, uint64_t words, SegArr* one, uint32_t n,
                            uint32_t* err)
{
    const uint64_t i0 = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x;
    for (uint64_t i = i0; i < words; i += (uint64_t)gridDim.x * blockDim.x) p[i] = 0;
    if (one && i0 == 0) {
        *one = SegArr{0, n, 0, 0, 0};
        *err = 0;
    }
}

// Digit counts of every key position of one tile, added to its array's; the last tile of
// the array makes the element starts and the rounds to run.  E: the rounds' tile.
template <int KB, int NT>
__global__ __launch_bounds__(NT) void k_seg_hist(SegArgs<KB, 0> a, uint32_t E)
{
    using K = typename UInt<KB>::T;
    constexpr uint32_t nt = KB, CLOG = KB == 4 ? 2 : 1;  // copies of the counts: by lane
    constexpr int U = 8;
    static_assert(NT / 64 >= nt, "one wave per key position");
    __shared__ uint32_t h[(nt * 256) << CLOG];
    __shared__ uint32_t last, mask;
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t tile = a.t0 + blockIdx.x, ai = a.map[tile];
    // Only where the host's and the device's offsets disagree: the tile's array is not one of
    // the group's, or was placed in another group's scratch.  Such an array is never counted
    // in full, so no round of it runs; the tile is handed to the group's first array, past
    // whose end the rounds find it.  (The same check in the rounds cost 1.5 us of 51.)
    const bool ours = ai - a.a0 < a.na;
    SegArr e{};
    if (ours) e = a.arr[ai];
    const uint32_t ti = tile - e.tile0, ntiles = (e.n + E - 1) / E;
    if (!ours || ti >= ntiles || e.group != a.group) {
        if (tid == 0) {
            a.map[tile] = a.a0;
            raise_error(a.err, kErrBounds);
        }
        return;
    }
    const uint32_t o = ti * E, cnt = min(E, e.n - o);
    const K* const src = a.Ak + e.o0 + o;
    for (uint32_t i = tid; i < (nt * 256) << CLOG; i += NT) h[i] = 0;
    if (tid == 0) mask = 0;
    __syncthreads();
    uint32_t* const mine = h + (lane & ((1u << CLOG) - 1));
    for (uint32_t c = 0; c < cnt; c += NT * U) {
        K x[U];
#pragma unroll
        for (int j = 0; j < U; j++) x[j] = src[min(c + j * NT + tid, cnt - 1)];
#pragma unroll
        for (int j = 0; j < U; j++) {
            if (c + j * NT + tid < cnt) {
#pragma unroll
                for (uint32_t t = 0; t < nt; t++)
                    atomicAdd(mine + ((t * 256 + ((uint32_t)(x[j] >> (8 * t)) & 0xFFu)) << CLOG), 1u);
            }
        }
    }
    __syncthreads();
    uint32_t* const hist = a.hist + (uint64_t)(ai - a.a0) * nt * 256;
    for (uint32_t i = tid; i < nt * 256; i += NT) {
        uint32_t s = 0;
#pragma unroll
        for (uint32_t c = 0; c < 1u << CLOG; c++) s += h[(i << CLOG) + c];
        if (s) add_agent(hist + i, s);
    }
    __builtin_amdgcn_s_waitcnt(0);  // this thread's additions are done
    __syncthreads();
    if (tid == 0) last = add_agent(a.arrived + (ai - a.a0), 1u) == ntiles - 1;
    __syncthreads();
    if (!last) return;
    if (wave < nt) {  // four digits per lane
        uint32_t x[4], s = 0;
        bool all = false;
#pragma unroll
        for (int k = 0; k < 4; k++) {
            x[k] = ld_agent(hist + wave * 256 + lane * 4 + k);
            all |= x[k] == e.n;
        }
#pragma unroll
        for (int k = 0; k < 4; k++) {
            const uint32_t t = x[k];
            x[k] = s;
            s += t;
        }
        const uint32_t before = wave_incl_scan(s) - s;
#pragma unroll
        for (int k = 0; k < 4; k++) hist[wave * 256 + lane * 4 + k] = before + x[k];
        if (ballot(all) == 0 && lane == 0) atomicOr(&mask, 1u << wave);
    }
    __syncthreads();
    if (tid == 0) {
        uint32_t m = mask;
        if (__popc(m) & 1) m |= ~m & (m + 1);  // n_t is even: some round is constant
        a.rounds[ai - a.a0] = m;
    }
}

// One round over the tiles of a group: see the top of this file, and k_tile_round for the
// ranks, the staging and what keeps the registers down.
template <int KB, int VB, class SH>
__global__ __launch_bounds__(SH::WAVES * 64)
__attribute__((amdgpu_waves_per_eu(SH::OCC))) void k_seg_round(SegArgs<KB, VB> a)
{
    using K = typename UInt<KB>::T;
    using V = typename Payload<VB>::T;
    constexpr int SMAX = 256, WAVES = SH::WAVES, ITEMS = SH::ITEMS;
    constexpr int NT = WAVES * 64, E = NT * ITEMS, SEG = 64 * ITEMS, DW = SMAX / 64;
    constexpr int SB = KB > VB ? KB : VB;
    constexpr bool OR_RANK = KB == 4 && VB <= 4 && E * SB >= WAVES * SMAX * 8;
    constexpr int SCH = 4, LBW = 8;
    constexpr uint32_t nt = KB;
    static_assert(SMAX <= NT && E <= 32768, "one digit per thread, 16-bit positions");
    __shared__ __align__(16) unsigned char stage[E * SB];
    K* const lk = (K*)stage;
    V* const lv = (V*)stage;
    __shared__ __align__(16) uint16_t wh[WAVES * SMAX];
    __shared__ uint32_t dt[SMAX], tmp[DW], claimed;
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;

    if (tid == 0) claimed = add_agent(a.ctr + a.r, 1u);
    __syncthreads();
    const uint32_t lt = claimed, tile = a.t0 + lt;  // claimed < grid = tiles of the group
    const uint32_t ai = a.map[tile], r = a.r, shift = 8 * r;
    const SegArr e = a.arr[ai];
    const uint32_t run = a.rounds[ai - a.a0];
    if (!(run >> r & 1u)) return;
    const bool back = __popc(run & ((1u << r) - 1)) & 1;  // from the scratch to the planes
    const uint32_t ti = tile - e.tile0;
    if ((uint64_t)ti * E >= e.n) {  // a tile that k_seg_hist found in no array of the group
        if (tid == 0) raise_error(a.err, kErrBounds);
        return;
    }
    const uint32_t o = ti * E, total = min((uint32_t)E, e.n - o);
    K* const pk = a.Ak + e.o0;
    K* const sk = a.Sk + (uint64_t)e.scr64 * 64;
    const K* const src = (back ? sk : pk) + o;
    K* const dstk = back ? pk : sk;
    const V* srcv = nullptr;
    V* dstv = nullptr;
    if constexpr (VB != 0) {
        V* const pv = a.Av + e.o0;
        V* const sv = a.Sv + (uint64_t)e.scr64 * 64;
        srcv = (back ? sv : pv) + o;
        dstv = back ? pv : sv;
    }

    K key[ITEMS];
    V val[ITEMS];
    const uint32_t s0 = wave * SEG + lane;
#pragma unroll
    for (int j = 0; j < ITEMS; j++) key[j] = src[min(s0 + j * 64, total - 1)];
    if constexpr (VB != 0) {
#pragma unroll
        for (int j = 0; j < ITEMS; j++) val[j] = srcv[min(s0 + j * 64, total - 1)];
    }
    const uint32_t mine = total > s0 ? min((uint32_t)ITEMS, (total - s0 + 63) / 64) : 0u;
    const uint32_t nvalid = mine == 32 ? ~0u : (1u << mine) - 1u;
    const bool wfull = ballot(mine != (uint32_t)ITEMS) == 0;
    const uint32_t d = tid;
    uint32_t start = 0;  // elements of the array with smaller digits
    if (d < SMAX) start = a.hist[((uint64_t)(ai - a.a0) * nt + r) * SMAX + d];

    uint16_t* const myh = wh + wave * SMAX;
    uint64_t* const myor = (uint64_t*)stage + wave * SMAX;
    for (uint32_t i = lane; i < SMAX / 2; i += 64) ((uint32_t*)myh)[i] = 0;
    if constexpr (OR_RANK)
        for (uint32_t i = lane; i < SMAX; i += 64) myor[i] = 0;
    uint32_t rp[ITEMS / 2];
    rank_wave<8, OR_RANK>(key, nvalid, wfull, shift, 8, myh, myor, rp);
    __syncthreads();

    // the tile's digit counts, published at once, and the wave offsets
    uint32_t* const row = a.state + (uint64_t)lt * SMAX;
    uint32_t c = 0;
    if (d < SMAX) {
#pragma unroll
        for (int i0 = 0; i0 < WAVES; i0 += 4) {
            uint32_t w[4];
#pragma unroll
            for (int i = 0; i < 4; i++) w[i] = wh[(i0 + i) * SMAX + d];
#pragma unroll
            for (int i = 0; i < 4; i++) {
                wh[(i0 + i) * SMAX + d] = (uint16_t)c;
                c += w[i];
            }
        }
        st_agent(row + d, c | seg_tag(r) | (ti ? kSegAgg : kSegIncl));
    }
    const uint32_t incl = wave_incl_scan(c);
    if (lane == 63 && wave < DW) tmp[wave] = incl;
    __syncthreads();
    uint32_t ex = incl - c;
    if (d < SMAX) {
#pragma unroll
        for (uint32_t w = 0; w < DW; w++) ex += w < wave ? tmp[w] : 0u;
#pragma unroll
        for (int i = 0; i < WAVES; i++) wh[i * SMAX + d] += (uint16_t)ex;
    }
    __syncthreads();

    // stage the keys in (digit, slot) order
    const uint16_t* const woff = wh + wave * SMAX;
    auto stage_keys = [&](auto full) {
        const uint32_t sh = opaque(shift);
#pragma unroll
        for (int j = 0; j < ITEMS; j++) {
            if (j % 4 == 0) __builtin_amdgcn_sched_barrier(0);
            uint32_t p = j & 1 ? rp[j / 2] >> 16 : rp[j / 2] & 0xFFFFu;
            if (full.value || p != 0xFFFFu) {
                p += woff[(uint32_t)(key[j] >> sh) & 0xFFu];
                lk[p] = key[j];
            }
            if (j & 1) rp[j / 2] = (rp[j / 2] & 0xFFFFu) | p << 16;
            else rp[j / 2] = (rp[j / 2] & 0xFFFF0000u) | p;
            pin(rp[j / 2]);
        }
    };
    if (wfull) stage_keys(std::true_type{});
    else stage_keys(std::false_type{});

    // look back over the array's earlier tiles, LBW at a time
    if (d < SMAX) {
        uint32_t acc = 0, k = ti, spins = 0;
        bool stalled = false;
        while (k > 0) {
            const uint32_t m = stalled ? 1u : min<uint32_t>(LBW, k);
            uint32_t w[LBW];
#pragma unroll
            for (int i = 0; i < LBW; i++)
                if ((uint32_t)i < m) w[i] = ld_agent(row + d - (uint64_t)(ti - k + 1 + i) * SMAX);
            uint32_t used = 0;
            bool ready = true, found = false;
#pragma unroll
            for (int i = 0; i < LBW; i++) {
                if ((uint32_t)i < m && ready && !found) {
                    if ((w[i] & kSegStatus) && (w[i] & kSegTag) == seg_tag(r)) {
                        acc += w[i] & kSegValue;
                        used = i + 1;
                        found = (w[i] & kSegStatus) == kSegIncl;
                    } else {
                        ready = false;
                    }
                }
            }
            k -= used;
            if (found) break;
            stalled = !ready && used == 0;
            if (!ready) {
                if (spin_give_up(++spins, a.err)) break;
                spin_pause();
            }
        }
        if (ti) st_agent(row + d, (acc + c) | seg_tag(r) | kSegIncl);
        dt[d] = start + acc - ex;
    }
    __syncthreads();

    // scatter: keys, then the payload staged in the same LDS
    uint32_t dst[VB ? ITEMS : 1];
    const bool tfull = total == (uint32_t)E;
    auto scatter_keys = [&](auto full) {
        const uint32_t sh = opaque(shift);
#pragma unroll
        for (int i = 0; i < ITEMS; i++) {
            if (i % SCH == 0) __builtin_amdgcn_sched_barrier(0);
            const uint32_t p = tid + i * NT;
            if (full.value || p < total) {
                const K k = lk[p];
                uint32_t pos = p + dt[(uint32_t)(k >> sh) & 0xFFu];
                if (pos >= e.n) {  // never for consistent digit starts
                    raise_error(a.err, kErrBounds);
                    pos = 0;
                }
                st_global(dstk + pos, k);
                if constexpr (VB != 0) {
                    dst[i] = pos;
                    pin(dst[i]);
                }
            }
        }
    };
    if (tfull) scatter_keys(std::true_type{});
    else scatter_keys(std::false_type{});
    if constexpr (VB != 0) {
        __syncthreads();  // every staged key was read
        auto stage_vals = [&](auto full) {
#pragma unroll
            for (int j = 0; j < ITEMS; j++) {
                if (j % SCH == 0) __builtin_amdgcn_sched_barrier(0);
                const uint32_t p = j & 1 ? rp[j / 2] >> 16 : rp[j / 2] & 0xFFFFu;
                if (full.value || p != 0xFFFFu) lv[p] = val[j];
            }
        };
        if (wfull) stage_vals(std::true_type{});
        else stage_vals(std::false_type{});
        __syncthreads();
        auto scatter_vals = [&](auto full) {
#pragma unroll
            for (int i = 0; i < ITEMS; i++) {
                if (i % SCH == 0) __builtin_amdgcn_sched_barrier(0);
                const uint32_t p = tid + i * NT;
                if (full.value || p < total) st_global(dstv + dst[i], lv[p]);
            }
        };
        if (tfull) scatter_vals(std::true_type{});
        else scatter_vals(std::false_type{});
    }
}

}  // namespace rs
