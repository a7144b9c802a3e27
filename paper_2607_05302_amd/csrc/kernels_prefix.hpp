// Digit starts of super-tiles: the count of each digit before every group of
// 2^st_log2 tiles of a round's input.  A tile of the round kernel then looks
// back only over the earlier tiles of its own super-tile, so no chain of
// look-backs runs across the whole launch.
//
// Slots follow the round kernel: slot s of the input is element (s mod b) of
// logical block sigma + floor(s / b), used when (s mod b) < blen of that block
// (Radsort), or element s of the array (out-of-place).  Super-tile u covers
// slots [u * 2^sts_log2, (u + 1) * 2^sts_log2).
#pragma once

#include "common.hpp"
#include "kernel_round.hpp"
#include "kernels_state.hpp"

namespace rs {

constexpr uint32_t kHistLog2 = 12;  // LDS words of digit counts per workgroup: 4096
constexpr int kHistWords = 1 << kHistLog2;
constexpr uint32_t kCopiesLog2 = 4;  // at most 16 copies of each count
constexpr int kMaxSuperBlocks = 2048;  // blocks of one super-tile held in LDS

// Exclusive sums down the columns of a[rows][sigma], in place, by one workgroup; the
// column totals go to total[sigma].  The rows come from other workgroups and the results go to others: agent-scope accesses.
// Several threads share a column, each a run of rows held in registers where it fits (32
// rows), so that their loads, one trip to memory, are in flight together.  part: LDS,
// max(NT, sigma) words.  Contains barriers.
template <int NT>
__device__ void scan_columns(uint32_t* a, uint32_t rows, uint32_t sigma, uint32_t* part,
                             uint32_t* total)
{
    constexpr uint32_t REG = 32;
    const uint32_t NP = sigma >= NT ? 1u : NT / sigma;  // threads per column
    const uint32_t per = (rows + NP - 1) / NP;
    const uint32_t tid = threadIdx.x;
    for (uint32_t i0 = 0; i0 < NP * sigma; i0 += NT) {
        const uint32_t i = i0 + tid, d = i % sigma, q0 = min(rows, (i / sigma) * per),
                       q1 = min(rows, q0 + per);
        const bool mine = i < NP * sigma;
        uint32_t x[REG], s = 0;
        for (uint32_t q = q0; mine && q < q1; q += REG) {
#pragma unroll
            for (uint32_t k = 0; k < REG; k++)
                x[k] = q + k < q1 ? ld_agent(a + (uint64_t)(q + k) * sigma + d) : 0u;
#pragma unroll
            for (uint32_t k = 0; k < REG; k++) s += x[k];
        }
        __syncthreads();  // part is free
        if (mine) part[i] = s;
        __syncthreads();
        uint32_t run = 0;
        for (uint32_t k = d + i0; mine && k < i; k += sigma) run += part[k];
        for (uint32_t q = q0; mine && q < q1; q += REG) {
            if (per > REG) {
#pragma unroll
                for (uint32_t k = 0; k < REG; k++)
                    x[k] = q + k < q1 ? ld_agent(a + (uint64_t)(q + k) * sigma + d) : 0u;
            }
#pragma unroll
            for (uint32_t k = 0; k < REG; k++) {
                if (q + k < q1) st_agent(a + (uint64_t)(q + k) * sigma + d, run);
                run += x[k];
            }
        }
        if (mine && i / sigma == NP - 1) {
            // a run past the end of the rows has added up everything before it
            st_agent(total + d, run);
        }
    }
}

// cnt[u * sigma + d] = elements with digit d in the super-tiles of u's chunk (kScanRows
// rows) before u, for every u of the grid (super-tiles past the input count as empty),
// and csum[c * sigma + d] = the same before chunk c, so that the digit start of
// super-tile u is cnt[u][d] + csum[u / kScanRows][d].  A workgroup counts one super-tile;
// the last one of a chunk to finish (counted in csum[c][0], zero on entry) scans the
// chunk's rows, and the last chunk (counter *done, zero on entry) scans the chunks and
// makes the round's plan from the digit totals, which also go to the last row, past the
// input (plan: 1; 2: with element starts; 3: packed, see plan_round).  One launch: a scan
// kernel of its own took 9 us at 2^24 elements and 12 us at 2^28.
//
// The counting is bound by the read of the keys.  Counts are kept in `copies` LDS tables
// laid out counter by counter (counter d of copy c at word d * copies + c), lane l adding
// to copy l mod copies: equal digits of a wave then meet in different words and banks.
// Measured per pass: 2^27 uint64 keys of 4096 skewed values 469 us with a table per wave,
// 246 us with 16 copies by lane (4.4 TB/s); 2^28 uniform uint64 keys 430 and 444 us; 4, 16
// and 32 copies are alike.
//
// A super-tile spans at most kMaxSuperBlocks blocks.
template <int KB, bool OOP, int NT>
__global__ __launch_bounds__(NT) void k_supertile_counts(
    const typename UInt<KB>::T* __restrict__ Ak, const typename UInt<KB>::T* __restrict__ Tk,
    const uint32_t* __restrict__ pi, const uint32_t* __restrict__ blen,
    const uint32_t* __restrict__ f_in_p, uint64_t n, uint32_t shift, uint32_t bits,
    uint32_t log2b, uint32_t npi, uint32_t sts_log2, uint32_t* __restrict__ cnt,
    uint32_t* __restrict__ csum, uint32_t* err, uint32_t* __restrict__ done, uint32_t plan,
    PlanPtrs pp)
{
    using K = typename UInt<KB>::T;
    constexpr uint32_t NW = NT / 64;
    constexpr int U = 16;  // loads in flight per thread
    __shared__ uint32_t h[kHistWords];
    __shared__ uint32_t bphys[OOP ? 1 : kMaxSuperBlocks], blen_s[OOP ? 1 : kMaxSuperBlocks];
    __shared__ uint32_t last, tmp[NT / 64];
    const uint32_t sigma = 1u << bits, dmask = sigma - 1, two_sigma = 2 * sigma;
    const uint32_t clog = min(kCopiesLog2, kHistLog2 - bits), copies = 1u << clog;
    const uint32_t tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    uint32_t* const mine = h + (lane & (copies - 1));
    for (uint32_t i = tid; i < copies * sigma; i += NT) h[i] = 0;

    const uint64_t s0 = (uint64_t)blockIdx.x << sts_log2, span = 1ull << sts_log2;
    const uint32_t b = 1u << log2b;
    auto add = [&](K x) { atomicAdd(mine + (((uint32_t)(x >> shift) & dmask) << clog), 1u); };
    if constexpr (OOP) {
        __syncthreads();
        const uint64_t s1 = min<uint64_t>(n, s0 + span);
        for (uint64_t c = s0; c < s1; c += (uint64_t)NT * U) {
            K x[U];
            if (c + (uint64_t)NT * U <= s1) {  // no checks
#pragma unroll
                for (int j = 0; j < U; j++) x[j] = Ak[c + j * NT + tid];
#pragma unroll
                for (int j = 0; j < U; j++) add(x[j]);
                continue;
            }
#pragma unroll
            for (int j = 0; j < U; j++) {
                const uint64_t sl = c + (uint64_t)j * NT + tid;
                x[j] = sl < s1 ? Ak[sl] : (K)0;
            }
#pragma unroll
            for (int j = 0; j < U; j++)
                if (c + (uint64_t)j * NT + tid < s1) add(x[j]);
        }
    } else {
        const uint32_t f_in = max(sigma, min(*f_in_p, npi));
        const uint32_t nblk = max(1u, (uint32_t)(span >> log2b));
        const uint32_t L0 = sigma + (uint32_t)(s0 >> log2b);
        for (uint32_t i = tid; i < nblk; i += NT) {
            const uint32_t L = L0 + i;
            uint32_t phys = 0, len = 0;
            if (L < f_in) {
                phys = pi[L];
                len = min(blen[L], b);
                if (phys >= npi) {  // never for a consistent state
                    raise_error(err, kErrBounds);
                    phys = 0;
                    len = 0;
                }
            }
            bphys[i] = phys;
            blen_s[i] = len;
        }
        __syncthreads();
        // each wave reads pieces of a block, at most U * 64 slots long
        const uint32_t plog = min<uint32_t>(log2b, 6 + 4);
        static_assert(U == 16, "pieces of 1024 slots");
        const uint32_t pieces = (uint32_t)(span >> plog);
        const uint32_t first = (uint32_t)s0 & (b - 1);  // 0 unless a block spans super-tiles
        for (uint32_t i = wave; i < pieces; i += NW) {
            const uint32_t at = first + (i << plog), bi = at >> log2b, o0 = at & (b - 1);
            const uint32_t len = __builtin_amdgcn_readfirstlane(blen_s[bi]);
            const uint32_t phys = __builtin_amdgcn_readfirstlane(bphys[bi]);
            const K* kp = blockat(Ak, Tk, phys, two_sigma, log2b);
            K x[U];
            if (o0 + U * 64 <= len) {  // a whole piece of 1024 elements: no checks
#pragma unroll
                for (int j = 0; j < U; j++) x[j] = kp[o0 + j * 64 + lane];
#pragma unroll
                for (int j = 0; j < U; j++) add(x[j]);
                continue;
            }
#pragma unroll
            for (int j = 0; j < U; j++) {
                const uint32_t o = o0 + j * 64 + lane;
                x[j] = (uint32_t)j * 64 < 1u << plog && o < len ? kp[o] : (K)0;
            }
#pragma unroll
            for (int j = 0; j < U; j++)
                if ((uint32_t)j * 64 < 1u << plog && o0 + j * 64 + lane < len) add(x[j]);
        }
    }
    __syncthreads();
    for (uint32_t d = tid; d < sigma; d += NT) {
        uint32_t s = 0;  // the copies from a start of this thread's own (banks)
        for (uint32_t c = 0; c < copies; c++) s += h[(d << clog) + ((c + d) & (copies - 1))];
        st_agent(cnt + (uint64_t)blockIdx.x * sigma + d, s);
    }
    // The rows pass between workgroups by agent-scope stores and loads: each thread waits
    // until its stores are done (a barrier waits for none of them), then one thread counts
    // the workgroup in.  (An agent-scope release fence here writes back the whole L2 in
    // every wave: 2.1 ms per pass at 2^28.)
    const uint32_t ch = blockIdx.x / kScanRows, r0 = ch * kScanRows;
    const uint32_t rows = min<uint32_t>(kScanRows, gridDim.x - r0);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (tid == 0) last = add_agent(csum + (uint64_t)ch * sigma, 1u) == rows - 1;
    __syncthreads();
    if (!last) return;
    uint32_t* const part = h;  // the counts were read
    static_assert(kHistWords >= NT && kHistWords >= 2048, "part holds max(NT, sigma) words");
    scan_columns<NT>(cnt + (uint64_t)r0 * sigma, rows, sigma, part, csum + (uint64_t)ch * sigma);
    const uint32_t chunks = (gridDim.x + kScanRows - 1) / kScanRows;
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (tid == 0) last = add_agent(done, 1u) == chunks - 1;
    __syncthreads();
    if (!last) return;
    scan_columns<NT>(csum, chunks, sigma, part, cnt + (uint64_t)(gridDim.x - 1) * sigma);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();  // the totals row is written by this workgroup; h is free
    const bool packed = plan == 3;
    static_assert(kHistWords >= 2 << 11, "h holds two arrays of sigma words, sigma up to 2^11");
    plan_round<NT>(cnt + (uint64_t)(gridDim.x - 1) * sigma, sigma, log2b, h, h + sigma, tmp, pp.S,
                   pp.Pidx, pp.Plen, pp.f, packed || plan == 2 ? pp.est : nullptr, packed);
}

// The plans of all rounds of a one-call sort at once: the digit counts of every key
// position (which do not depend on the order of the elements) added up in est, zero on entry,
// by one pass over the keys; the last workgroup (counter *arrived, zero on entry) turns them
// into S, P, f and est of every round and the rounds' modes, one wave per round.  Counts by
// lane copies as in k_supertile_counts.  sigma <= 256.
// Bound by the read of the keys while a key has four digits: 0.27 ms at 2^28 uint32
// (4.0 TB/s), where counting before each round took 4 x 0.27 ms; 0.50 ms at 2^28 uint64
// (4.3 TB/s) against 8 x 0.43 ms.
constexpr uint32_t kPlanWords = 16384;  // LDS words of counts
template <int KB, int FB, int NT>
__global__ __launch_bounds__(NT) void k_hist_plan(const typename UInt<KB>::T* __restrict__ keys,
                                                  uint64_t n, uint32_t bits_, uint32_t nt_,
                                                  uint32_t log2b, uint32_t per_wg, PlanPtrs p,
                                                  uint32_t* __restrict__ mode,
                                                  uint32_t* __restrict__ arrived)
{
    using K = typename UInt<KB>::T;
    constexpr int U = 8;
    constexpr uint32_t NW = NT / 64;
    __shared__ uint32_t h[kPlanWords], last, vary[2];
    const uint32_t bits = FB ? (uint32_t)FB : bits_, nt = FB ? (8u * KB + FB - 1) / (FB ? FB : 1) : nt_;
    const uint32_t sigma = 1u << bits, dmask = sigma - 1, words = nt * sigma;
    uint32_t clog = 0;  // copies: 16 (8 for 64-bit keys), fewer where few keys are counted
    while (clog < kCopiesLog2 && (words << (clog + 1)) <= min(kPlanWords, per_wg / 4)) clog++;
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (uint32_t i = tid; i < words << clog; i += NT) h[i] = 0;
    if (tid < 2) vary[tid] = 0;
    __syncthreads();
    uint32_t* const mine = h + (lane & ((1u << clog) - 1));
    const uint64_t c0 = (uint64_t)blockIdx.x * per_wg, c1 = min<uint64_t>(n, c0 + per_wg);
    for (uint64_t c = c0; c < c1; c += NT * U) {
        K x[U];
#pragma unroll
        for (int j = 0; j < U; j++) x[j] = keys[min<uint64_t>(c + j * NT + tid, c1 - 1)];
#pragma unroll
        for (int j = 0; j < U; j++) {
            if (c + j * NT + tid < c1)
#pragma unroll
                for (uint32_t r = 0; r < nt; r++)
                    atomicAdd(mine + ((r * sigma + ((uint32_t)(x[j] >> (bits * r)) & dmask)) << clog),
                              1u);
        }
    }
    __syncthreads();
    for (uint32_t i = tid; i < words; i += NT) {
        uint32_t s = 0;
        for (uint32_t c = 0; c < 1u << clog; c++) s += h[(i << clog) + c];
        if (s) add_agent(p.est + i, s);
    }
    __builtin_amdgcn_s_waitcnt(0);  // this thread's additions are done
    __syncthreads();
    if (tid == 0) last = add_agent(arrived, 1u) == gridDim.x - 1;
    __syncthreads();
    if (!last) return;
    // the rounds whose digit varies (bit r of vary)
    uint32_t* const cnt = h;  // the totals
    for (uint32_t i = tid; i < words; i += NT) cnt[i] = ld_agent(p.est + i);
    __syncthreads();
    for (uint32_t r = wave; r < nt; r += NW) {
        bool all = false;
        for (uint32_t d = lane; d < sigma; d += 64) all |= cnt[r * sigma + d] == n;
        if (ballot(all) == 0 && lane == 0) atomicOr(&vary[r >> 5], 1u << (r & 31));
    }
    __syncthreads();
    const uint64_t v = (uint64_t)vary[1] << 32 | vary[0];
    const uint32_t top = v ? 63u - (uint32_t)__builtin_clzll(v) : nt - 1;
    const uint32_t b = 1u << log2b;
    for (uint32_t r = wave; r < nt; r += NW) {
        const bool packed = r == top;
        uint32_t elems = 0, blocks = 0;  // before this group of 64 digits
        for (uint32_t d0 = 0; d0 < sigma; d0 += 64) {
            const uint32_t d = d0 + lane;
            const bool in = d < sigma;
            const uint32_t c = in ? cnt[r * sigma + d] : 0u;
            const uint32_t ei = wave_incl_scan(c), es = elems + ei - c;
            const uint32_t span = c + (packed ? es & (b - 1) : 0u);
            const uint32_t C = in ? 1 + (span >> log2b) : 0u;
            const uint32_t bi = wave_incl_scan(C), s = sigma + blocks + bi - C;
            if (in) {
                p.S[r * sigma + d] = s;
                p.Pidx[(r + 1) * sigma + d] = s + C - 1;
                p.Plen[(r + 1) * sigma + d] = span & (b - 1);
                p.est[r * sigma + d] = es;
            }
            elems += (uint32_t)__builtin_amdgcn_readlane((int)ei, 63);
            blocks += (uint32_t)__builtin_amdgcn_readlane((int)bi, 63);
        }
        if (lane == 0) {
            p.f[r + 1] = sigma + blocks;
            mode[r] = packed ? kModePacked : v >> r & 1u ? kModeRun : kModeSkip;
        }
    }
}

}  // namespace rs
