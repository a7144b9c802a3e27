// The Radsort round (Alg. 5) in the default draw order for digits of at most 8
// bits: the protocol of kernel_round.hpp (tiles, super-tile look-back, ring, pool
// draws, the GPU form of Lemma 1: see there; one-call sorts: CHAIN below), arranged so that two workgroups with
// large tiles share a compute unit.
//
// What bounds it: a tile is a chain of dependent steps (claim, block table, loads,
// ranks, look-back, draws, first blocks, two scatters), several of them round
// trips to memory.  One workgroup per compute unit leaves the memory idle during
// the other steps; so the tile's state is cut down until two tiles of the large
// shape fit a compute unit (128 registers per lane, 80 KB of LDS each):
//  - one digit per thread: the digit's counts, starts and draw numbers stay in that
//    thread's registers (no LDS arrays);
//  - ranks are 16-bit, two per register, and become the staged positions; the
//    digit is taken from the key again where it is needed;
//  - per-wave digit counts are 16-bit;
//  - the thread that learns a block's place writes its addresses straight into the
//    pointer table.
#pragma once

#include "common.hpp"
#include "kernel_round.hpp"
#include "kernels_state.hpp"

namespace rs {

// the smallest block the kernel takes: a tile then writes at most E / 1024 + 2 sigma
// blocks, which keeps the pointer table small
constexpr uint32_t kTileMinLog2b = 10;

// Hides a value's origin from the optimiser: what is computed from it is computed
// again in the next phase instead of being held in registers across it.
__device__ __forceinline__ uint32_t opaque(uint32_t x)
{
    asm volatile("" : "+s"(x));
    return x;
}

// Keeps the computation of x where it is written (not sunk to x's use, which would
// hold its inputs instead).
__device__ __forceinline__ void pin(uint32_t& x) { asm volatile("" : "+v"(x)); }

// Stable rank of every element of a wave among the wave's elements of the same digit, in
// slot order (item j of all lanes before item j + 1), two 16-bit ranks per word of rp
// (0xFFFF: no element; nvalid bit j: item j of this lane holds one; wfull: all of them
// do).  myh: the wave's digit counts, zero on entry, complete on return; myor: its OR
// table, zero on entry (OR only).  items: the items looked at, a multiple of G; the rest are
// empty and their words of rp left as they are.
template <int FB, bool OR, int G = 1, typename K, int ITEMS>
__device__ __forceinline__ void rank_wave(const K (&key)[ITEMS], uint32_t nvalid, bool wfull,
                                          uint32_t shift, uint32_t bits, uint16_t* myh,
                                          uint64_t* myor, uint32_t (&rp)[ITEMS / 2],
                                          int items = ITEMS)
{
    const uint32_t lane = lane_id(), dmask = (1u << bits) - 1;
    // Lanes with the same digit as this one, found bit by bit on the vector unit, or
    // through the wave's OR table: each lane ORs its bit into the word of its digit
    // and reads the word back.  Lower lanes of the set come first (slot order); the
    // highest one commits the set's count.
    auto match = [&](uint32_t dw, uint64_t vm) {
        uint32_t lo = (uint32_t)vm, hi = (uint32_t)(vm >> 32);
#pragma unroll
        for (uint32_t k = 0; k < (FB ? FB : 8); k++) {
            if (FB || k < bits) {
                // nb: all ones where the lane's bit k is set; its peers are the lanes
                // whose bit is the same: p & ~(ballot ^ nb)
                const uint32_t nb = (uint32_t)__builtin_amdgcn_sbfe((int)dw, k, 1);
                const uint64_t bk = ballot(nb != 0);
                lo = __builtin_amdgcn_bitop3_b32(lo, (uint32_t)bk, nb, 0x90);
                hi = __builtin_amdgcn_bitop3_b32(hi, (uint32_t)(bk >> 32), nb, 0x90);
            }
        }
        return (uint64_t)hi << 32 | lo;
    };
    auto commit = [&](uint32_t dg, uint64_t peers, bool clear) {
        const uint32_t old = myh[dg];
        if ((peers >> lane) == 1ull) {  // highest lane of the set
            myh[dg] = (uint16_t)(old + (uint32_t)__popcll(peers));
            if (clear) myor[dg] = 0;
        }
        return old + popc_below(peers);
    };
    auto put_rank = [&](int j, uint32_t r) {
        if (j & 1) rp[j / 2] |= r << 16;
        else rp[j / 2] = r;
        pin(rp[j / 2]);
    };
    auto by_ballot = [&](auto full, int from) {
#pragma unroll
        for (int j = 0; j < ITEMS; j++) {
            if (j < from) continue;
            if (j % G == 0 && j >= items) break;
            if constexpr (ITEMS >= 32) __builtin_amdgcn_sched_barrier(0);  // registers
            const uint32_t dw = (uint32_t)(key[j] >> shift);
            uint32_t r = 0xFFFFu;
            if constexpr (full.value) {
                r = commit(dw & dmask, match(dw, ~0ull), false);
            } else {
                const bool valid = nvalid >> j & 1u;
                const uint64_t peers = match(dw, ballot(valid));
                if (valid) r = commit(dw & dmask, peers, false);
            }
            put_rank(j, r);
        }
    };
    if (!wfull) {
        by_ballot(std::false_type{}, 0);
    } else if constexpr (!OR) {
        by_ballot(std::true_type{}, 0);
    } else {
        // the first item tells a wave of skewed digits (six or more equal ones), whose
        // table accesses would serialise
        const uint32_t dw0 = (uint32_t)(key[0] >> shift);
        const uint64_t peers0 = match(dw0, ~0ull);
        put_rank(0, commit(dw0 & dmask, peers0, false));
        if (ballot(__popcll(peers0) >= 6) != 0) {
            by_ballot(std::true_type{}, 1);
        } else {
            const uint64_t mybit = 1ull << lane;
#pragma unroll
            for (int j = 1; j < ITEMS; j++) {
                if (j % G == 0 && j >= items) break;
                if constexpr (ITEMS >= 32) __builtin_amdgcn_sched_barrier(0);  // registers
                const uint32_t dg = (uint32_t)(key[j] >> shift) & dmask;
                __hip_atomic_fetch_or(myor + dg, mybit, __ATOMIC_RELAXED,
                                      __HIP_MEMORY_SCOPE_WORKGROUP);
                const uint64_t peers = myor[dg];
                put_rank(j, commit(dg, peers, true));
            }
        }
    }
}

// CHAIN: how a tile finds its digit starts.
//  kChainNone: the counting pass before the round gives those of its super-tile, and it adds
//    the counts of the super-tile's earlier tiles (rounds planned one at a time).
// One-call sorts plan all rounds ahead (k_hist_plan) and run no counting pass; a tile looks
// back over all earlier tiles, each of which publishes its counts and then its counts up to
// and including itself:
//  kChainRows: a word of its own for every (tile, digit), 0 until published; n < 2^30;
//  kChainRing: 64-bit words in a ring, tagged with their tile.  Tile T takes the slot of
//    T - W (W slots) once T - W and T - W + 1 are done: then T - W writes it no more, and a
//    reader that still wants its word starts its look-back again and meets the inclusive
//    count of T - W + 1, or a later one, first.
// A finished look-back over all earlier tiles also says that all of them have published
// their counts, hence that their loads have returned: the tile's draws wait for nothing
// more.  Measured without and with, whole sorts: 7.39 -> 6.47 ms at 2^28 uint32 pairs,
// 13.8 -> 12.6 ms at 2^28 skewed uint64, 5.93 -> 4.82 ms at 2^26 uint64+uint32 (a counting
// pass reads the keys and their block table again each round: 270, 429 and 157 us); rows:
// 0.81 -> 0.75 ms at 2^24 uint32 pairs, 0.42 -> 0.34 ms at 2^20 uint64+uint32.
constexpr int kChainNone = 0, kChainRows = 1, kChainRing = 2;
constexpr uint32_t kRowAgg = 1u << 30, kRowIncl = 2u << 30, kRowValue = kRowAgg - 1;
constexpr uint64_t kRingAgg = 1ull << 62, kRingIncl = 2ull << 62;
// status | tile + 1 (30 bits) | value
__device__ __forceinline__ uint64_t ring_word(uint64_t status, uint32_t tile, uint32_t value)
{
    return status | (uint64_t)(tile + 1) << 32 | value;
}

template <int KB, int VB, int FB, class SH, int CHAIN>
__global__ __launch_bounds__(SH::WAVES * 64)
__attribute__((amdgpu_waves_per_eu(SH::OCC))) void k_tile_round(TileArgs<KB, VB> a)
{
    using K = typename UInt<KB>::T;
    using V = typename Payload<VB>::T;
    constexpr int SMAX = 256;
    constexpr int WAVES = SH::WAVES, ITEMS = SH::ITEMS;
    constexpr int NT = WAVES * 64, E = NT * ITEMS, SEG = 64 * ITEMS;
    constexpr int MAXBLK = E >> kTileMinLog2b;  // blocks a tile reads
    constexpr int TBL = MAXBLK + 2 * SMAX;      // blocks a tile can write
    constexpr int POOL = MAXBLK + SMAX;         // blocks a tile can draw
    constexpr int SB = KB > VB ? KB : VB;
    // Ranks by OR table where the digits of a wave are spread (4-byte keys, records of at
    // most 8 bytes: the LDS unit has room), else by ballots, which cost the same whatever
    // the digits are.  Measured at 2^28 uniform uint32 + uint32: 1.240 ms per round with
    // the table, 1.284 ms with ballots; 2^28 uniform uint64 1.417 and 1.414 ms; 2^27
    // uint64 keys of 4096 skewed values 0.743 and 0.572 ms.
    constexpr bool OR_RANK = KB == 4 && VB <= 4;
    constexpr int SCH = 4;  // items of a loop scheduled together (bounds the registers)
    // Predecessors read per look-back step.  Ring words cost traffic: at 2^28 uint32 pairs a
    // round took 1238, 1288, 1336 and 1358 us with 1, 2, 4 and 8 of them; keys alone have
    // shorter tiles, so longer look-backs: 889, 875, 880 and 904 us at 2^28 uint32.
    constexpr int LBW = CHAIN == kChainRing ? (VB ? 1 : 2)
                        : CHAIN == kChainRows || E < 16384 ? 8 : 4;
    static_assert(SMAX <= NT, "one digit per thread");
    static_assert((E & (E - 1)) == 0 && E <= 32768, "16-bit positions, 0xFFFF unused");
    static_assert(MAXBLK >= 1 && MAXBLK <= NT, "one thread per block of a tile");
    static_assert(!OR_RANK || E * SB >= WAVES * SMAX * 8, "OR tables live in the stage");
    static_assert(ITEMS % 2 == 0, "two ranks per register");

    const uint32_t bits = FB ? (uint32_t)FB : a.bits;
    const uint32_t sigma = 1u << bits, dmask = sigma - 1;
    const uint32_t log2b = a.log2b, b = 1u << log2b, two_sigma = 2 * sigma;
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;

    // OR tables, then the keys in (digit, slot) order, then the payload
    __shared__ __align__(16) unsigned char stage[E * SB];
    K* const lk = (K*)stage;
    V* const lv = (V*)stage;
    __shared__ __align__(16) uint16_t wh[WAVES * SMAX];  // wave counts, then wave offsets
    __shared__ uint64_t ptab[(VB ? 2 : 1) * TBL];        // addresses of the blocks written
    __shared__ uint2 dt[SMAX];                           // (rank offset, table offset)
    __shared__ uint32_t pool[POOL];                      // physical blocks of the draws
    __shared__ uint32_t bphys[MAXBLK], blen[MAXBLK];
    constexpr int DW = SMAX / 64;  // waves that own digits
    __shared__ uint32_t tmp[2 * DW], claimed;

    const uint32_t wlog = a.ring_log2;
    const uint64_t wmask = (1ull << wlog) - 1;
    const uint32_t mst = 1u << a.st_log2;  // tiles per super-tile

    bool packed = false;
    if constexpr (CHAIN != kChainNone) {
        const uint32_t m = *a.mode;
        if (m == kModeSkip) return;  // the round's digit is the same for every element
        packed = m == kModePacked;
    }

    // ---- claim a tile; its blocks ----------------------------------------------------
    if (tid == 0) claimed = add_agent(a.tile_ctr, 1u);
    // f is clamped so that a corrupt state can never index past pi
    const uint32_t f_in = max(sigma, min(*a.f_in, a.npi));
    const uint64_t nslots = (uint64_t)(f_in - sigma) << log2b;
    const uint32_t ntiles = (uint32_t)((nslots + E - 1) / E);
    __syncthreads();
    const uint32_t tile = claimed;
    if (tile >= ntiles) return;
#ifdef RS_TIMELINE
    if (tid == 0 && a.tl) a.tl[(uint64_t)tile * kTlStamps + 15] = __builtin_amdgcn_s_memrealtime();
#endif
    const uint64_t slot0 = (uint64_t)tile * E;
    const uint32_t nblk = (E >> log2b) ? (E >> log2b) : 1u;
    if (tid < nblk) {
        const uint32_t L = sigma + (uint32_t)(slot0 >> log2b) + tid;
        uint32_t phys = 0, len = 0;
        if (L < f_in) {
            phys = a.pi_old[L];
            len = min(a.blen[L], b);
            if (phys >= a.npi) {  // never for a consistent state; read nothing
                raise_error(a.err, kErrBounds);
                phys = 0;
                len = 0;
            }
        }
        bphys[tid] = phys;
        blen[tid] = len;
    }
    __syncthreads();
    RS_STAMP(0);

    // ---- load: item j of a wave is 64 consecutive slots of one block (b >= 1024).  Every
    // slot of a block is loaded, used or not (blocks are whole in memory): no branches
    K key[ITEMS];
    V val[ITEMS];
    static_assert(ITEMS <= 32, "validity bits");
    const uint32_t ws0 = wave * SEG + ((uint32_t)slot0 & (b - 1) & ~(uint32_t)(E - 1));
    constexpr int PER = 1 << (kTileMinLog2b - 6);  // items of 1024 slots, always of one block
#pragma unroll
    for (int j0 = 0; j0 < ITEMS; j0 += PER) {
        const uint32_t s = ws0 + j0 * 64;
        const uint32_t phys = __builtin_amdgcn_readfirstlane(bphys[s >> log2b]);
        const uint32_t off0 = (s & (b - 1)) + lane;
        const K* kb = blockat(a.Ak, a.Tk, phys, two_sigma, log2b) + off0;
#pragma unroll
        for (int j = 0; j < PER && j0 + j < ITEMS; j++) key[j0 + j] = kb[j * 64];
        if constexpr (VB != 0) {
            const V* vb = blockat(a.Av, a.Tv, phys, two_sigma, log2b) + off0;
#pragma unroll
            for (int j = 0; j < PER && j0 + j < ITEMS; j++) val[j0 + j] = vb[j * 64];
        }
    }
    // bit j: slot j of this lane holds an element (all of them but in a few waves)
    uint32_t nvalid = 0;
#pragma unroll 1
    for (int j = 0; j < ITEMS; j++) {
        const uint32_t s = ws0 + j * 64;
        nvalid |= (s & (b - 1)) + lane < blen[s >> log2b] ? 1u << j : 0u;
    }
    const bool wfull = ballot(nvalid != (ITEMS == 32 ? ~0u : (1u << ITEMS) - 1u)) == 0;

    // per-digit data of the round, for the thread that owns the digit
    const uint32_t d = tid;
    uint32_t Sd = 0, sbase = 0, poff = 0;
    if (d < sigma) {
        Sd = a.S[d];
        if constexpr (CHAIN == kChainNone) sbase = super_start(a, tile >> a.st_log2, sigma, d);
        if (packed) poff = a.pack_est[d] & (b - 1);  // the packed round's offset
    }
    // reuse of this tile's ring slot: the done words of the tiles that must have
    // finished, requested now and checked before the counts are published
    uint32_t rq = 0, rqend = 0, rv = 0;
    const uint32_t W64 = 1u << (wlog - 1);  // kChainRing's slots
    if (CHAIN == kChainRing ? tile >= W64 : CHAIN == kChainNone && (uint64_t)tile > wmask) {
        if constexpr (CHAIN == kChainRing) {
            rq = tile - W64;
            rqend = rq + 2;
        } else {
            rq = tile - (uint32_t)wmask - 1;            // tile - W
            rqend = min((rq | (mst - 1)) + 1, ntiles);  // end of its super-tile
        }
        if (rq + tid < rqend) rv = ld_agent(a.done + ((rq + tid) & wmask));
    }

    // ---- stable rank among equal digits of the wave ----------------------------------
    uint16_t* const myh = wh + wave * SMAX;
    uint64_t* const myor = (uint64_t*)stage + wave * SMAX;
    for (uint32_t i = lane; i < SMAX / 2; i += 64) ((uint32_t*)myh)[i] = 0;
    if constexpr (OR_RANK)
        for (uint32_t i = lane; i < SMAX; i += 64) myor[i] = 0;
    uint32_t rp[ITEMS / 2];  // ranks, later staged positions; 0xFFFF: no element
    rank_wave<FB, OR_RANK>(key, nvalid, wfull, a.shift, bits, myh, myor, rp);
    for (uint32_t j = rq + tid; j < rqend; j += NT) {
        const uint32_t* w = a.done + (j & wmask);
        uint32_t v = j == rq + tid ? rv : ld_agent(w), spins = 0;
        while (v <= j) {
            if (spin_give_up(++spins, a.err)) break;
            spin_pause();
            v = ld_agent(w);
        }
    }
    // Every load of the tile has returned (the payload is not read before staging, so
    // wait for it here): from the counts' publication on, other tiles may reuse the
    // tile's blocks.
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    RS_STAMP(1);
#ifdef RS_DEBUG_ORDER
    // ordering check: see kernel_round.hpp
    if (a.consumed && b <= (uint32_t)E) {
        const uint32_t L = sigma + (uint32_t)(slot0 >> log2b) + tid;
        if (tid < nblk && L < f_in) st_agent(a.consumed + bphys[tid], a.tag_mark);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        __syncthreads();
    }
#endif

    // ---- the tile's digit counts (published at once), wave offsets --------------------
    const uint32_t st0 = tile & ~(mst - 1);  // first tile of this tile's super-tile
    uint32_t c = 0;                          // elements of digit d
    if (d < sigma) {
        // four waves at a time (registers: the records are live)
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
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (CHAIN == kChainRows)
            st_agent(a.rows + (uint64_t)tile * sigma + d, c | (tile ? kRowAgg : kRowIncl));
        else if constexpr (CHAIN == kChainRing)
            st_agent(a.ring64 + (uint64_t)(tile & (W64 - 1)) * sigma + d,
                     ring_word(tile ? kRingAgg : kRingIncl, tile, c));
        else if (mst > 1)  // a super-tile of one tile has no look-back
            st_agent(a.agg + (uint64_t)(tile & wmask) * sigma + d, c | epoch_bit(tile, wlog));
    }
    const uint32_t cincl = wave_incl_scan(c);
    if (lane == 63 && wave < DW) tmp[wave] = cincl;
    __syncthreads();
    uint32_t ex = cincl - c, total = 0;  // elements of the tile with smaller digits
#pragma unroll
    for (uint32_t w = 0; w < DW; w++) {
        const uint32_t t = tmp[w];
        ex += w < wave ? t : 0u;
        total += t;
    }
    if (d < sigma) {
#pragma unroll
        for (int i = 0; i < WAVES; i++) {
            wh[i * SMAX + d] += (uint16_t)ex;
            if (i % 4 == 3) __builtin_amdgcn_sched_barrier(0);
        }
    }
    RS_STAMP(2);

    // ---- look back over the super-tile -------------------------------------------------
    uint32_t bs = sbase + poff;  // digit-d elements before the tile (from the block starts)
    if constexpr (CHAIN != kChainNone) {
        if (d < sigma) {
            using Wd = typename std::conditional<CHAIN == kChainRows, uint32_t, uint64_t>::type;
            auto word = [&](uint32_t t) -> Wd* {
                if constexpr (CHAIN == kChainRows) return a.rows + (uint64_t)t * sigma + d;
                else return a.ring64 + (uint64_t)(t & (W64 - 1)) * sigma + d;
            };
            uint32_t k = tile, spins = 0, acc = 0;
            bool stalled = false;
            while (k > 0) {
                const uint32_t m = stalled ? 1u : min<uint32_t>(LBW, k);
                Wd w[LBW];
#pragma unroll
                for (int i = 0; i < LBW; i++)
                    if ((uint32_t)i < m) w[i] = ld_agent(word(k - 1 - i));
                uint32_t used = 0;
                bool ready = true, found = false, again = false;
#pragma unroll
                for (int i = 0; i < LBW; i++) {
                    if ((uint32_t)i < m && ready && !found) {
                        if constexpr (CHAIN == kChainRows) {
                            ready = w[i] != 0;
                            found = w[i] >= kRowIncl;
                            if (ready) acc += w[i] & kRowValue;
                        } else {
                            const uint32_t tag = (uint32_t)(w[i] >> 32) & 0x3FFFFFFFu;
                            ready = tag == k - i;            // tile k - 1 - i
                            again = tag > k - i;             // its slot was taken over
                            found = ready && w[i] >= kRingIncl;
                            if (ready) acc += (uint32_t)w[i];
                        }
                        if (ready) used = i + 1;
                    }
                }
                k -= used;
                if (found) break;
                if (again) {
                    k = tile;
                    acc = 0;
                }
                stalled = !ready && used == 0 && !again;
                if (!ready) {
                    if (spin_give_up(++spins, a.err)) break;
                    spin_pause();
                }
            }
            if constexpr (CHAIN == kChainRows) {
                if (tile) st_agent(word(tile), (acc + c) | kRowIncl);
            } else {
                if (tile) st_agent(word(tile), ring_word(kRingIncl, tile, acc + c));
                __builtin_amdgcn_s_waitcnt(0);  // before the tile is done (ring reuse)
            }
            bs += acc;
        }
    } else if (d < sigma) {
        // the counts of tiles st0 .. tile-1, up to LBW loads at once; while
        // one has not published, poll that one alone
        uint32_t k = tile, spins = 0;
        bool stalled = false;
        while (k > st0) {
            const uint32_t m = stalled ? 1u : min<uint32_t>(LBW, k - st0);
            uint32_t w[LBW];
#pragma unroll
            for (int i = 0; i < LBW; i++)
                if ((uint32_t)i < m)
                    w[i] = ld_agent(a.agg + (uint64_t)((k - 1 - i) & wmask) * sigma + d);
            uint32_t used = 0;
            bool ready = true;
#pragma unroll
            for (int i = 0; i < LBW; i++) {
                if ((uint32_t)i < m && ready) {
                    if ((w[i] & ~kCntMask) == epoch_bit(k - 1 - i, wlog)) {
                        bs += w[i] & kCntMask;
                        used = i + 1;
                    } else {
                        ready = false;
                    }
                }
            }
            k -= used;
            stalled = !ready && used == 0;
            if (!ready) {
                if (spin_give_up(++spins, a.err)) break;
                spin_pause();
            }
        }
    }

    // ---- block draws -------------------------------------------------------------------
    // the block a draw names: Eq. 1, or one of the packed round's extra blocks
    auto out_block = [&](auto* A, auto* T, auto* X, uint32_t j) {
        return j < a.npi ? blockat(A, T, j, two_sigma, log2b)
                         : X + ((uint64_t)(j - a.npi) << log2b);
    };
    auto put_block = [&](uint32_t e, uint32_t phys) {
        if (phys >= a.npi_x) {  // never for a consistent state: send the writes to T
            raise_error(a.err, kErrBounds);
            phys = 0;
        }
        if constexpr (VB != 0) {
            ptab[2 * e] = (uint64_t)(uintptr_t)out_block(a.Ak, a.Tk, a.Xk, phys);
            ptab[2 * e + 1] = (uint64_t)(uintptr_t)out_block(a.Av, a.Tv, a.Xv, phys);
        } else {
            ptab[e] = (uint64_t)(uintptr_t)out_block(a.Ak, a.Tk, a.Xk, phys);
        }
    };
    const uint32_t q0 = bs >> log2b;
    const uint32_t nfill = d < sigma ? ((bs + c) >> log2b) - q0 : 0u;
    const uint32_t nwrite = c ? ((bs + c - 1) >> log2b) - q0 + 1 : 0u;
    // request the block that takes the digit's first elements (drawn by an earlier
    // tile) now; it is used after this tile's own draws are out
    uint32_t first = kEmpty;
    if (c) {
        if (q0 == 0) first = a.pi_old[d];
        else if (Sd + q0 < a.npi_x) first = ld_agent(a.pi_new + Sd + q0);
    }
    // F: draws made by earlier tiles; nfills: draws of this tile; the scans of the
    // blocks each digit draws (low half) and writes (high half; both sums < 2^16)
    const uint32_t fw = nfill | nwrite << 16, fwincl = wave_incl_scan(fw);
    const uint32_t qsum = wave_sum(d < sigma ? q0 : 0u);
    __syncthreads();  // tmp was read; the look-back of every digit is done
    if (CHAIN != kChainRows && tid == 0) st_agent(a.done + (tile & wmask), tile + 1);
    if (lane == 63 && wave < DW) {
        tmp[wave] = qsum;
        tmp[DW + wave] = fwincl;
    }
    __syncthreads();
    RS_STAMP(4);
    uint32_t F = 0, nfills = 0, fwbo = fwincl - fw;
#pragma unroll
    for (uint32_t w = 0; w < DW; w++) {
        F += tmp[w];
        const uint32_t t = tmp[DW + w];
        nfills += t & 0xFFFFu;
        fwbo += w < wave ? t : 0u;
    }
    const uint32_t fbo = fwbo & 0xFFFFu, tbo = fwbo >> 16;  // for digits' owners (wave < DW)
    RS_STAMP(10);
    // Request the pool entries of the draws, and the done words of the earlier tiles
    // whose input blocks they are.  Draw k of the round takes pool entry k: the input
    // block sigma + k (logical), or in the packed round the extra block npi + k for
    // k < sigma and then the input block k.
    auto pool_entry = [&](uint32_t k) -> uint32_t {
        if (packed) return k < sigma ? a.npi + k : (k < a.npi ? a.pi_old[k] : a.npi_x);
        const uint32_t h = sigma + k;
        return h < a.npi ? a.pi_old[h] : a.npi_x;
    };
    uint32_t pv = 0;
    if (tid < nfills) pv = pool_entry(F + tid);
    // The drawn blocks of this super-tile were loaded before their tiles' counts, which
    // the look-back read; for earlier tiles wait until they are done.  The wait ends
    // before the draws are published: later tiles that continue a drawn block write
    // into it as soon as they see its entry in pi_new.
    if (CHAIN == kChainNone && nfills) {
        const uint32_t olo = (uint32_t)(((uint64_t)F << log2b) / E);
        const uint32_t ohi =
            min<uint32_t>((uint32_t)((((uint64_t)(F + nfills) << log2b) - 1) / E) + 1, st0);
        for (uint32_t o = olo + tid; o < ohi; o += NT) {
            const uint32_t* w = a.done + (o & wmask);
            uint32_t v = ld_agent(w), spins = 0;
            while (v <= o) {
                if (spin_give_up(++spins, a.err)) break;
                spin_pause();
                v = ld_agent(w);
            }
        }
    }
    if (tid < nfills) pool[tid] = pv;  // nfills <= E / b + sigma <= NT
    __syncthreads();
    RS_STAMP(11);
#ifdef RS_DEBUG_ORDER
    // ordering check: every drawn block that holds input of this round must be marked
    if (a.consumed && b <= (uint32_t)E) {
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        for (uint32_t i = tid; i < nfills; i += NT) {
            const uint32_t phys = pool[i], h = packed ? F + i : sigma + F + i;
            if (h >= sigma && h < f_in && phys < a.npi && ld_agent(a.consumed + phys) != a.tag)
                raise_error(a.err, kErrOrder);
        }
    }
#endif
    // publish the tile's draws
    for (uint32_t i = 1; i <= nfill; i++) {
        const uint32_t L = Sd + q0 + i, r = fbo + i - 1;
        uint32_t phys = r < (uint32_t)POOL ? pool[r] : a.npi_x;
        if (phys < a.npi_x && L < a.npi_x) st_agent(a.pi_new + L, phys);
        else phys = a.npi_x;  // put_block reports it
        if (i < nwrite) put_block(tbo + i, phys);
        else if (phys >= a.npi_x) raise_error(a.err, kErrBounds);
    }
    RS_STAMP(12);

    // ---- stage the keys in (digit, slot) order -----------------------------------------
    RS_STAMP(13);
    const uint16_t* const woff = wh + wave * SMAX;
    auto stage_keys = [&](auto full) {
        const uint32_t shift = opaque(a.shift);
#pragma unroll
        for (int j = 0; j < ITEMS; j++) {
            if (j % 4 == 0) __builtin_amdgcn_sched_barrier(0);
            uint32_t p = j & 1 ? rp[j / 2] >> 16 : rp[j / 2] & 0xFFFFu;
            if (full.value || p != 0xFFFFu) {
                p += woff[(uint32_t)(key[j] >> shift) & dmask];
                lk[p] = key[j];
            }
            if (j & 1) rp[j / 2] = (rp[j / 2] & 0xFFFFu) | p << 16;
            else rp[j / 2] = (rp[j / 2] & 0xFFFF0000u) | p;
            pin(rp[j / 2]);
        }
    };
    if (wfull) stage_keys(std::true_type{});
    else stage_keys(std::false_type{});
    RS_STAMP(3);

    // ---- the block of each digit's first elements --------------------------------------
    if (d < sigma) {
        if (c) {
            if (Sd + q0 >= a.npi_x) {  // never for a consistent state
                first = a.npi_x;
            } else {
                uint32_t spins = 0;
                while (first == kEmpty) {
                    if (spin_give_up(++spins, a.err)) break;
                    spin_pause();
                    first = ld_agent(a.pi_new + Sd + q0);
                }
            }
            put_block(tbo, first);
        }
        dt[d] = make_uint2(bs - ex, tbo - q0);
    }
    __syncthreads();
    RS_STAMP(5);
    RS_STAMP(6);

    // ---- scatter: keys first, remembering (table entry, offset) of each position; then
    // the payload is staged in the same LDS and follows its key
    uint32_t dst[VB ? ITEMS : 1];
    const bool tfull = total == (uint32_t)E;  // the same for the workgroup
    auto scatter_keys = [&](auto full) {
#pragma unroll
        for (int i = 0; i < ITEMS; i++) {
            if (i % SCH == 0) __builtin_amdgcn_sched_barrier(0);
            const uint32_t p = tid + i * NT;
            if (full.value || p < total) {
                const K k = lk[p];
                const uint2 x = dt[(uint32_t)(k >> a.shift) & dmask];
                const uint32_t r = p + x.x;
                const uint32_t e = x.y + (r >> log2b);
                const uint32_t off = r & (b - 1);
                st_global((K*)(uintptr_t)ptab[(VB ? 2 : 1) * e] + off, k);
                if constexpr (VB != 0) {
                    dst[i] = e << 16 | off;  // e < TBL, off < b <= 2^16
                    pin(dst[i]);
                }
            }
        }
    };
    if (tfull) scatter_keys(std::true_type{});
    else scatter_keys(std::false_type{});
    if constexpr (VB != 0) {
        __syncthreads();  // every staged key was read
        RS_STAMP(7);
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
        RS_STAMP(8);
        auto scatter_vals = [&](auto full) {
#pragma unroll
            for (int i = 0; i < ITEMS; i++) {
                if (i % SCH == 0) __builtin_amdgcn_sched_barrier(0);
                const uint32_t p = tid + i * NT;
                if (full.value || p < total)
                    st_global((V*)(uintptr_t)ptab[2 * (dst[i] >> 16) + 1] + (dst[i] & 0xFFFFu),
                              lv[p]);
            }
        };
        if (tfull) scatter_vals(std::true_type{});
        else scatter_vals(std::false_type{});
    }
#ifdef RS_TIMELINE
    __builtin_amdgcn_s_waitcnt(0);
#endif
    RS_STAMP(9);
}

}  // namespace rs
