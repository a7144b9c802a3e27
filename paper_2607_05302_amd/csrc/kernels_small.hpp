// Sorting small arrays whole on chip: one workgroup sorts one array in LDS and
// registers, so it needs no extra device memory at all.  This is the regime the paper
// hands to an out-of-place sort (arrays smaller than T, Sec. 5).
//
// Workgroup i takes array i (elements [offsets[i], offsets[i+1]) of the key and payload
// planes) and sorts it if it has lo < n <= E elements; with offsets null the one array of n1
// elements.  With a claim counter (zero on entry) the workgroups claim the `step` residue
// classes of the indices modulo `step` one after another, look at a class's arrays with one
// lane each, and sort those of their size: an array of another size costs a lane and not a
// claim, and neighbours of one size fall to different workgroups.  An array is dealt out over
// all the waves, ceil(n / NT) items to a lane (slot s = wave * 64 items + j * 64 + lane).
// Each round is the stable counting sort of Alg. 1 on 8 bits: ranks within the waves by the OR
// table or by ballots (rank_wave), digit and wave starts by scans, the records to LDS at start
// + rank and back in slot order.  A round whose digit is the same for every element is left out.
//
// What bounds it: the latency of a round's steps (ranks of `items` items, the barriers, two
// scans) and, with many arrays, the instructions of the ranks.  So a short array takes few
// items per lane and a small workgroup; the large shape takes its items G at a time, without a
// branch between them, so that their LDS accesses are in flight together (a branch per item
// also held 128 registers, two workgroups to a compute unit; 84 now), and ranks by the OR table
// unless the keys are 8 bytes without payload, whose registers it would need.  The payload is
// staged in the keys' bytes after them.  Per batch, with a branch per item and ballots / now:
// 20 000 uint32 pairs arrays of 8192 records 1602 / 1372 us, of 3000 877 / 812 us; of 4096
// records of 16 bytes 1757 / 1559 us; G = 4, 2 there 1504, 1479 us by ballots; one array of
// 1500 pairs 37.1 / 35.6 us (the copy of the input and the wait for the stream included;
// 290 us through the general path).
#pragma once

#include "common.hpp"
#include "kernel_tile.hpp"

namespace rs {

template <int KB, int VB, int WAVES, int ITEMS, bool CLAIM>
__global__ __launch_bounds__(WAVES * 64) __attribute__((amdgpu_waves_per_eu(4))) void k_sort_small(
    typename UInt<KB>::T* keys, typename Payload<VB>::T* vals, const uint64_t* offsets,
    uint32_t nseg, uint64_t n1, uint32_t lo, uint32_t* err, uint32_t* claim, uint32_t step)
{
    using K = typename UInt<KB>::T;
    using V = typename Payload<VB>::T;
    constexpr int NT = WAVES * 64, E = NT * ITEMS, SMAX = 256, DW = SMAX / 64;
    static_assert(NT >= SMAX, "one digit per thread");
    static_assert(E <= 32768, "16-bit positions");
    constexpr bool OR_RANK = WAVES == 8 && !(KB == 8 && VB == 0);
    constexpr int G = WAVES == 8 ? ITEMS / 4 : 1;  // items taken together
    static_assert(!OR_RANK || sizeof(K) * E >= WAVES * SMAX * 8, "OR tables live in the stage");
    // the keys in sorted order, then the payload in the same bytes
    __shared__ __align__(16) unsigned char stage[E * (KB > VB ? KB : VB)];
    K* const lk = (K*)stage;
    V* const lv = (V*)stage;
    __shared__ __align__(16) uint16_t wh[WAVES * SMAX];
    __shared__ uint32_t tmp[DW];
    __shared__ uint64_t vary;
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (!offsets && blockIdx.x == 0 && tid == 0 && err) *err = 0;  // the call's error word

    // the workgroup's own array, or the arrays of one class after another
    __shared__ uint32_t claimed;
    const bool many = CLAIM && step < nseg;  // classes of several arrays
    uint32_t cls = blockIdx.x;
    do {
    if constexpr (CLAIM) {
        __syncthreads();  // the class before is done
        if (tid == 0) claimed = add_agent(claim, 1u);
        __syncthreads();
        cls = claimed;
    }
    if (cls >= step) return;
    for (uint64_t i0 = cls; i0 < (CLAIM ? nseg : cls + 1); i0 += 64ull * step) {
    uint64_t left = 1;  // the arrays of this size among 64 of the class, the same in every wave
    if (many) {
        const uint64_t i = i0 + (uint64_t)lane * step;
        uint64_t len = 0;
        if (i < nseg) {
            const uint64_t first = offsets[i], end = offsets[i + 1];
            len = end > first ? end - first : 0;
        }
        left = ballot(len > max(lo, 1u) && len <= (uint64_t)E);
    }
    for (; left; left &= left - 1) {
    const uint64_t i = i0 + (uint64_t)__builtin_ctzll(left) * step;
    uint64_t o0 = 0, n64 = n1;
    if (CLAIM || offsets) {
        o0 = offsets[i];
        const uint64_t o1 = offsets[i + 1];
        n64 = o1 > o0 ? o1 - o0 : 0;
    }
    if (n64 <= max(lo, 1u) || n64 > (uint64_t)E) continue;  // nothing to do, or another's
    const uint32_t n = (uint32_t)n64;
    const int items = (int)((n + NT * G - 1) / (NT * G)) * G;
    const uint32_t s0 = wave * 64 * items + lane;
    K* const kp = keys + o0;
    V* vp = nullptr;
    if constexpr (VB != 0) vp = vals + o0;
    if (tid == 0) vary = 0;

    K key[ITEMS];
    V val[ITEMS];
    uint32_t nvalid = 0;
    const K ref = kp[0];
    K diff = 0;
#pragma unroll
    for (int j = 0; j < ITEMS; j++) {
        key[j] = 0;
        if (j < items && s0 + j * 64 < n) {
            key[j] = kp[s0 + j * 64];
            if constexpr (VB != 0) val[j] = vp[s0 + j * 64];
            nvalid |= 1u << j;
        }
    }
#pragma unroll
    for (int j = 0; j < ITEMS; j++)
        if (nvalid >> j & 1u) diff |= key[j] ^ ref;
    __syncthreads();
    if (diff) atomicOr((unsigned long long*)&vary, (unsigned long long)diff);
    __syncthreads();
    const uint64_t bits_vary = vary;  // bits in which the keys differ
    if (!bits_vary) continue;         // all equal: the array is sorted
    const bool wfull = ballot(nvalid != (1u << items) - 1u) == 0;
    // f of every item the lane holds, G without a branch in a wave whose items are all there
    auto each = [&](auto f) {
#pragma unroll
        for (int j0 = 0; j0 < ITEMS; j0 += G) {
            if (j0 >= items) break;
            if (wfull) {
#pragma unroll
                for (int j = j0; j < j0 + G; j++) f(j);
            } else {
#pragma unroll
                for (int j = j0; j < j0 + G; j++)
                    if (nvalid >> j & 1u) f(j);
            }
        }
    };

    for (uint32_t shift = 0; shift < 8 * KB; shift += 8) {
        if (!(bits_vary >> shift & 0xFFu)) continue;
        uint16_t* const myh = wh + wave * SMAX;
        uint64_t* const myor = (uint64_t*)stage + wave * SMAX;
        if constexpr (OR_RANK) {
            __syncthreads();  // the stage was read
            for (uint32_t i = lane; i < SMAX; i += 64) myor[i] = 0;
        }
        for (uint32_t i = lane; i < SMAX / 2; i += 64) ((uint32_t*)myh)[i] = 0;
        uint32_t rp[ITEMS / 2];
#pragma unroll
        for (int j = 0; j < ITEMS / 2; j++) rp[j] = ~0u;
        rank_wave<8, OR_RANK, G>(key, nvalid, wfull, shift, 8, myh, myor, rp, items);
        __syncthreads();
        uint32_t c = 0;
        if (tid < SMAX) {
#pragma unroll
            for (int w = 0; w < WAVES; w++) {
                const uint32_t t = wh[w * SMAX + tid];
                wh[w * SMAX + tid] = (uint16_t)c;
                c += t;
            }
        }
        const uint32_t incl = wave_incl_scan(c);
        if (lane == 63 && wave < DW) tmp[wave] = incl;
        __syncthreads();
        if (tid < SMAX) {
            uint32_t ex = incl - c;
#pragma unroll
            for (uint32_t w = 0; w < DW; w++) ex += w < wave ? tmp[w] : 0u;
#pragma unroll
            for (int w = 0; w < WAVES; w++) wh[w * SMAX + tid] += (uint16_t)ex;
        }
        __syncthreads();
        each([&](int j) {
            uint32_t p = j & 1 ? rp[j / 2] >> 16 : rp[j / 2] & 0xFFFFu;
            p += myh[(uint32_t)(key[j] >> shift) & 0xFFu];
            lk[p] = key[j];
            if constexpr (VB != 0)
                rp[j / 2] = j & 1 ? (rp[j / 2] & 0xFFFFu) | p << 16 : (rp[j / 2] & 0xFFFF0000u) | p;
        });
        __syncthreads();
        each([&](int j) { key[j] = lk[s0 + j * 64]; });
        if constexpr (VB != 0) {
            __syncthreads();
            each([&](int j) { lv[j & 1 ? rp[j / 2] >> 16 : rp[j / 2] & 0xFFFFu] = val[j]; });
            __syncthreads();
            each([&](int j) { val[j] = lv[s0 + j * 64]; });
        }
    }
    each([&](int j) {
        kp[s0 + j * 64] = key[j];
        if constexpr (VB != 0) vp[s0 + j * 64] = val[j];
    });
    }
    }
    } while (CLAIM);
}

}  // namespace rs
