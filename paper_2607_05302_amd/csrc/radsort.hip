// Host side of the Radsort library: argument checks, workspace layout, the
// launch sequence of Alg. 2 on a HIP stream, and the C ABI of include/radsort.h.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <new>
#include <utility>
#include <vector>

#include "../../include/radsort.h"
#include "common.hpp"
#include "kernels_state.hpp"
#include "kernel_round.hpp"
#include "kernel_seg.hpp"
#include "kernel_tile.hpp"
#include "kernels_prefix.hpp"
#include "kernels_small.hpp"
#include "kernels_wg.hpp"
#include "kernels_finalize.hpp"
#include "kernels_finalize_seq.hpp"

using namespace rs;

namespace {

thread_local hipError_t g_last_hip = hipSuccess;
#ifdef RS_TIMELINE
uint64_t* g_tl = nullptr;  // stamps of the Radsort round kernel (timeline builds)
uint64_t g_tl_tiles = 0;
#endif
// statistics and phase events of the last sort call, per host thread
thread_local radsort_stats g_stats{};

#define RS_HIP(call)                                 \
    do {                                             \
        hipError_t e_ = (call);                      \
        if (e_ != hipSuccess) {                      \
            g_last_hip = e_;                         \
            return RADSORT_E_DEVICE;                 \
        }                                            \
    } while (0)

constexpr uint32_t kRingWords = 1u << 19;  // look-back ring: 2^ring_log2 * sigma count words
constexpr uint32_t kSuperSlotsLog2 = 16;   // slots per super-tile: 2^16 (8 tiles of 8192)

uint64_t align_up(uint64_t x, uint64_t a) { return (x + a - 1) / a * a; }

int ilog2(uint64_t x)
{
    int r = 0;
    while ((1ull << r) < x) r++;
    return r;
}

// Shape of the round kernel's workgroup per record size (KB key bytes, VB payload
// bytes), digit width (WIDE: more than 8 bits) and round (OOP: Alg. 1).  E = 64 *
// WAVES * ITEMS slots per tile.  The shape decides how many workgroups share a
// compute unit: the staged tile and per-wave digit counts must fit its 160 KB of
// LDS, the records held in registers its register file.
//   shape 0: one workgroup per CU, the next tile's records loaded into registers
//     while the current one is processed (PF), the payload staged beside the keys;
//   shape 1: two workgroups per CU (at most 128 VGPRs and about 68 KB of LDS
//     each): no register prefetch, the payload staged after the keys are written
//     out (SPLIT).  Measured at 2^28 uint32 + uint32, b = 2048: Radsort round
//     1.59 ms against 2.07 ms for shape 0, with one workgroup per tile;
//   shapes 2-4 (tiles of 4096 slots, two to three workgroups per CU) measured
//     slower (2.10-2.42 ms against 1.56 ms for shape 1, the same day), shapes
//     5-6 (16 waves of 8 slots) spill registers;
//     they are kept for measurement only (RS_ROUND_CFG selects a shape at build
//     time, RS_RADSORT_FORM the launch form of the Radsort round).
// The out-of-place round keeps shape 0 (1.50 ms, against 2.36 ms with shape 1).
#ifndef RS_ROUND_CFG
#define RS_ROUND_CFG 1
#endif
template <int KB, int VB, bool WIDE, bool OOP = false> struct TileCfg {
    static constexpr int C = (WIDE || OOP) ? 0 : RS_ROUND_CFG;
    static constexpr bool BIG = KB + VB >= 12;
    static constexpr bool NARROW = KB == 4 && VB <= 4;  // 8 bytes or less per record
    static constexpr int WAVES = WIDE ? 4 : (C == 3 ? 4 : C >= 5 ? 16 : 8);
    static constexpr int ITEMS = C == 0 ? (BIG ? 8 : 16)
                               : C == 1 ? (NARROW ? 16 : 8)
                               : C == 3 ? (BIG ? 8 : 16)
                               : C >= 5 ? 8
                                        : 8;
    static constexpr bool PF = C == 0 || C == 4;
    static constexpr bool SPLIT = C != 0;
    static constexpr int OCC = C == 0 ? 1 : C == 2 ? 6 : C == 5 ? 8 : C == 6 ? 6 : 4;
    using Shape = RoundShape<WAVES, ITEMS, PF, SPLIT, OCC>;
    static constexpr int E = 64 * WAVES * ITEMS;
};

// k_round's tile for large arrays of records of at most 8 bytes: shape 1
// with twice the slots per lane (4-byte keys: 16384-slot tiles; 8-byte keys without
// payload: 8192), one workgroup per compute unit.  Its digit runs per tile are twice
// as long and the super-tiles half as many.  Measured with 8-bit digits (b >= 1024 and
// the default draw order now run k_tile_round instead): uint32 +
// uint32 at 2^28, b = 2048, 8.20-8.27 ms per sort against 8.47 ms with the smaller
// tile (from 2^25 to 2^27 elements no faster: fewer tiles in flight, so it is taken
// from kLargeTileMin on); uint64 keys at b = 4096, 18.8 against 19.6 ms at 2^28 and
// 76.5 against 81.1 ms at 2^30.
template <int KB> struct LargeTile {  // KB = 4: keys of 4 bytes; 8: keys of 8 bytes, no payload
    static constexpr int WAVES = 8, ITEMS = KB == 4 ? 32 : 16;
    using Shape = RoundShape<WAVES, ITEMS, false, true, 2>;
    static constexpr int E = 64 * WAVES * ITEMS;
};
constexpr uint64_t kLargeTileMin = 1ull << 28;  // elements

// Tiles of k_tile_round (the default draw order, digits of at most 8 bits, blocks of
// 1024 elements or more).  Two workgroups share a compute unit with either tile; the
// large one holds 16384 slots (4-byte keys, records of at most 8 bytes) or 8192, so
// that a digit's run in a tile is 64 or 32 elements long (256 bytes).  Time per round,
// small tile against large one, uniform keys: uint32 pairs 32.0 / 35.3 us at 2^21, 46.6 /
// 43.1 at 2^22, 105 / 95 at 2^24, 417 / 323 at 2^26; uint64 + uint32 27.5 / 26.7 us at
// 2^20, 146 / 121 at 2^24, 708 / 498 at 2^26; uint64 keys 24.2 / 23.5 us at 2^20, 531 / 391 at
// 2^26: hence tile_large_min.  At 2^28 uint32 pairs, b = 2048, the large tile takes
// 1.240 ms per round (3.46 TB/s) against 1.536 ms for one workgroup per compute unit of
// the same tile in k_round (2.80 TB/s).
template <int KB, int VB, bool LARGE> struct TileShape {
    static constexpr bool NARROW = KB == 4 && VB <= 4;
    static constexpr int WAVES = 8;
    static constexpr int ITEMS = (NARROW ? 16 : 8) << (LARGE ? 1 : 0);
    using Shape = RoundShape<WAVES, ITEMS, false, true, 4>;
    static constexpr int E = 64 * WAVES * ITEMS;
};
constexpr uint64_t tile_large_min(uint32_t kb, uint32_t vb)
{
    return kb == 4 && vb <= 4 ? 1ull << 22 : 1ull << 20;
}
template <bool LARGE> uint32_t tile_shape_elems(uint32_t kb, uint32_t vb)
{
    return kb == 4 && vb <= 4 ? TileShape<4, 4, LARGE>::E : TileShape<8, 8, LARGE>::E;
}

struct Geo {
    uint64_t n = 0;
    uint32_t kb = 0, vb = 0, bits = 0, sigma = 0, nt = 0, b = 0, log2b = 0;
    uint64_t nb = 0;
    uint32_t npi = 0, E = 0, tiles = 0, ring_w = 0, ring_log2 = 0;
    uint32_t st_log2 = 0;                 // tiles per super-tile: 2^st_log2
    uint32_t supers = 0, oop_supers = 0;  // super-tiles of a Radsort / out-of-place round
    uint32_t lay_supers = 0;              // the super-tiles the workspace is laid out for
    uint32_t oop_E = 0, oop_st_log2 = 0;  // tile and super-tile of the out-of-place round
    bool fin_temps = false;       // finalize scratch holds the two-kernel F1's temporary blocks
    bool fin_temps_pack = false;  // the same for a packed state (n_pi + sigma blocks)
    bool large_tile = false;      // the Radsort round runs LargeTile (E = 16384)
    bool tile = false;            // the Radsort round is k_tile_round
    bool tile_large = false;      // ... with its large tile
};

// Workspace regions (byte offsets), each 256-byte aligned.
struct Layout {
    uint64_t Tk, Tv, pi0, pi1, blen, opened, S, Pidx, Plen, f, est, ctr, ring, agg, done,
        csum, stcnt, fin, alt_k, alt_v;
    uint64_t Xk, Xv, pack;  // a packed last round only: sigma extra blocks, bucket table
    uint64_t consumed;  // ordering-check builds only: a tag per physical block
    uint64_t zero, zero_bytes;  // what each round finds zeroed: ring, counters, chunk sums
    uint64_t fin_bytes, total;
};

template <bool WIDE, bool OOP> uint32_t tile_elems_t(uint32_t kb, uint32_t vb)
{
    if (kb == 4 && vb == 0) return TileCfg<4, 0, WIDE, OOP>::E;
    if (kb == 4 && vb == 4) return TileCfg<4, 4, WIDE, OOP>::E;
    if (kb == 4 && vb == 8) return TileCfg<4, 8, WIDE, OOP>::E;
    if (kb == 8 && vb == 0) return TileCfg<8, 0, WIDE, OOP>::E;
    if (kb == 8 && vb == 4) return TileCfg<8, 4, WIDE, OOP>::E;
    return TileCfg<8, 8, WIDE, OOP>::E;
}

// digits of more than 8 bits take the wide tile (per-wave counts of 2^11 digits)
uint32_t tile_elems(uint32_t kb, uint32_t vb, uint32_t bits, bool oop)
{
    if (bits > 8) return oop ? tile_elems_t<true, true>(kb, vb) : tile_elems_t<true, false>(kb, vb);
    return oop ? tile_elems_t<false, true>(kb, vb) : tile_elems_t<false, false>(kb, vb);
}

// Compute units of the current device; 256 (an MI355X) when no device answers.
uint32_t device_cus()
{
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        cus <= 0) {
        (void)hipGetLastError();
        return 256;
    }
    return (uint32_t)cus;
}

// Bytes of the round's counting state: the look-back count words, the digit starts of
// `supers` super-tiles (and a row of totals), and their chunk sums.
uint64_t count_word_bytes(const Geo& g) { return 4ull * g.sigma * g.ring_w; }
uint64_t digit_start_bytes(const Geo& g, uint64_t supers)
{
    return align_up(4ull * g.sigma * (supers + 1), 256);
}
uint64_t csum_bytes(const Geo& g, uint64_t supers)
{
    return align_up(4ull * g.sigma * ((supers + kScanRows) / kScanRows), 256);
}

int make_geo(Geo& g, uint64_t n, int key_bytes, int payload_bytes, int digit_bits,
             const radsort_opts* opts)
{
    if (key_bytes != 4 && key_bytes != 8) return RADSORT_E_INVALID;
    if (payload_bytes != 0 && payload_bytes != 4 && payload_bytes != 8) return RADSORT_E_INVALID;
    if (digit_bits < 1 || digit_bits > 16) return RADSORT_E_INVALID;
    // 12 .. 16 bits: 2 sigma b head-block elements, waves * sigma LDS counts and
    // digit runs shorter than a line per tile cost more than the round they save
    if (digit_bits > 11) return RADSORT_E_UNSUPPORTED;
#ifndef RS_DEBUG_ORDER
    if (opts && (opts->flags & RADSORT_F_DEBUG_ORDER)) return RADSORT_E_UNSUPPORTED;
#endif
    uint32_t b = (opts && opts->block_elems) ? opts->block_elems : 1024u;
    if (b < 64 || b > 65536 || (b & (b - 1))) return RADSORT_E_INVALID;
    if (n >= (1ull << 32)) return RADSORT_E_UNSUPPORTED;
    g.n = n;
    g.kb = key_bytes;
    g.vb = payload_bytes;
    g.bits = digit_bits;
    g.sigma = 1u << digit_bits;
    g.nt = (8 * key_bytes + digit_bits - 1) / digit_bits;
    g.b = b;
    g.log2b = ilog2(b);
    g.nb = n >> g.log2b;
    uint64_t npi = g.nb + 2ull * g.sigma;  // state table, Sec. 2.1
    // pi entries are 32-bit with the top bit free; finalize scans at most 4096^2 entries
    if (npi >= (uint64_t)kScanTile * kScanTile) return RADSORT_E_UNSUPPORTED;
    g.npi = (uint32_t)npi;
    g.large_tile = digit_bits <= 8 && n >= kLargeTileMin &&
                   ((key_bytes == 4 && payload_bytes <= 4) || (key_bytes == 8 && payload_bytes == 0));
    g.E = !g.large_tile ? tile_elems(g.kb, g.vb, g.bits, false)
          : key_bytes == 4 ? (uint32_t)LargeTile<4>::E : (uint32_t)LargeTile<8>::E;
    const uint32_t seq_E = g.E;  // the tile of the sequential draw order
    g.tile = digit_bits <= 8 && g.log2b >= kTileMinLog2b &&
             !(opts && (opts->flags & RADSORT_F_SEQ_DRAWS));
    if (g.tile) {
        g.tile_large = n >= tile_large_min(g.kb, g.vb);
        g.E = g.tile_large ? tile_shape_elems<true>(g.kb, g.vb) : tile_shape_elems<false>(g.kb, g.vb);
    }
    g.oop_E = tile_elems(g.kb, g.vb, g.bits, true);
#ifdef RS_DEBUG_ORDER
    if (opts && (opts->flags & RADSORT_F_DEBUG_ORDER) && g.b > g.E) return RADSORT_E_UNSUPPORTED;
#endif
    // input slots of a round: at most (floor(n/b) + sigma) blocks of b
    uint64_t slots = (g.nb + g.sigma) << g.log2b;
    g.tiles = (uint32_t)((slots + g.E - 1) / g.E);
    // ring slots (a power of two): one per tile when the tiles fit, else the cap;
    // with a slot per tile no slot is ever reused.  The ring and the super-tiles are
    // laid out for the smaller tile of the two draw orders, so that one workspace
    // serves both.
    const uint32_t lay_E = std::min(g.E, seq_E);
    const uint32_t lay_tiles = (uint32_t)((slots + lay_E - 1) / lay_E);
    const uint32_t ring_cap = std::max<uint32_t>(256u, kRingWords / g.sigma);
    uint32_t ring_w = 32;
    while (ring_w < lay_tiles && ring_w < ring_cap) ring_w <<= 1;
    g.ring_w = ring_w;
    g.ring_log2 = ilog2(g.ring_w);
    // a super-tile spans at least 2^kSuperSlotsLog2 slots and at least one block
    auto super_log2 = [&](uint32_t E) {
        const uint32_t elog = (uint32_t)ilog2(E);
        return std::max<uint32_t>(kSuperSlotsLog2 > elog ? kSuperSlotsLog2 - elog : 0u,
                                  g.log2b > elog ? g.log2b - elog : 0u);
    };
    const uint32_t lay_st = super_log2(lay_E);
    g.lay_supers = (lay_tiles + (1u << lay_st) - 1) >> lay_st;
    // One tile per super-tile (no look-back, and a counting pass of many small
    // workgroups) where its rows fit the memory laid out for the ring and the larger
    // super-tiles' rows; else super-tiles of at least 2^kSuperSlotsLog2 slots.  At
    // 2^20 uint32 pairs super-tiles of 2^16 slots were 17 workgroups: 20 us per pass.
    // Look-back words in the rows' place hold counts of up to kRowValue.
    g.st_log2 = n <= kRowValue &&
                        digit_start_bytes(g, g.tiles) + csum_bytes(g, g.tiles) <=
                        count_word_bytes(g) + csum_bytes(g, g.lay_supers) +
                            digit_start_bytes(g, g.lay_supers)
                    ? 0u
                    : super_log2(g.E);
    g.supers = (g.tiles + (1u << g.st_log2) - 1) >> g.st_log2;
    g.oop_st_log2 = super_log2(g.oop_E);
    const uint64_t oop_tiles = (n + g.oop_E - 1) / g.oop_E;
    g.oop_supers = (uint32_t)((oop_tiles + (1u << g.oop_st_log2) - 1) >> g.oop_st_log2);
    // F1 of finalize runs cooperatively on one workgroup per compute unit unless the
    // GPU is shared or that grid cannot cover the state; only the other form needs
    // temporary blocks in the workspace
    const bool shared = opts && (opts->flags & RADSORT_F_SHARED);
    const uint32_t cus = device_cus();
    g.fin_temps = shared || !fin_coop(g.npi, g.b, g.kb + g.vb, cus).covers;
    // the packed last round: its finalize is F1 over n_pi + sigma blocks, then the
    // spare blocks' slots copied into place (no compaction)
    g.fin_temps_pack = shared || !fin_coop(g.npi + g.sigma, g.b, g.kb + g.vb, cus).covers;
    return RADSORT_OK;
}

// Finalize scratch (parallel Alg. 7): see kernels_finalize.hpp.
uint64_t finalize_bytes(const Geo& g, bool pack)
{
    return fin_scratch_bytes(g.npi + (pack ? g.sigma : 0u), g.n, g.b, g.kb + g.vb,
                             pack ? g.fin_temps_pack : g.fin_temps);
}

// pack: the workspace of a sort whose last round is packed (one-call sorts): sigma
// extra blocks, and the block permutations and finalize arrays over n_pi + sigma
// blocks.  The small arrays come first, so that the error word's place depends
// on n_t and sigma only.
Layout make_layout(const Geo& g, bool oop, bool pack = false)
{
    Layout L{};
    uint64_t o = 0;
    auto take = [&](uint64_t bytes) {
        uint64_t at = o;
        o = align_up(o + bytes, 256);
        return at;
    };
    const uint64_t sig = g.sigma, nt = g.nt;
    pack = pack && !oop;
    L.S = take(4 * nt * sig);
    L.Pidx = take(4 * (nt + 1) * sig);
    L.Plen = take(4 * (nt + 1) * sig);
    L.f = take(4 * (nt + 1));
    L.est = take(4 * nt * sig);
    L.ctr = take(4 * (nt + 8));
    if (!oop) {
        const uint64_t npx = g.npi + (pack ? sig : 0);
        L.Tk = take(2 * sig * g.b * g.kb);
        L.Tv = take(2 * sig * g.b * g.vb);
        L.pi0 = take(4ull * npx);
        L.pi1 = take(4ull * npx);
        L.blen = take(4ull * npx);
        L.opened = take(8ull * g.sigma);
        if (pack) {
            L.Xk = take(sig * g.b * g.kb);
            L.Xv = take(sig * g.b * g.vb);
            L.pack = take(4 * (2 * sig + 2));
        }
    } else {
        L.alt_k = take(g.n * g.kb);
        L.alt_v = take(g.n * g.vb);
    }
#ifdef RS_DEBUG_ORDER
    L.consumed = oop ? 0 : take(4ull * g.npi);
#endif
    // the look-back ring (count words, done words), the tile counter of the round kernel
    // and the counter of the counting kernel, the chunk sums of the super-tile scan, zeroed
    // before each round; then the super-tile digit starts, with one more row for the
    // digit totals.  Finalize reuses all of it.
    const uint64_t supers = oop ? g.oop_supers : g.supers;
    const uint64_t lay_supers = oop ? g.oop_supers : g.lay_supers;
    const uint64_t done_bytes = align_up(4ull * g.ring_w + 8, 256);
    L.fin_bytes = oop ? 0 : finalize_bytes(g, pack);
    L.ring = take(std::max(count_word_bytes(g) + done_bytes + csum_bytes(g, lay_supers) +
                               digit_start_bytes(g, lay_supers),
                           L.fin_bytes));
    if (!oop && g.st_log2 == 0) {
        // no count words: the digit starts take their place (make_geo checks the room)
        L.stcnt = L.agg = L.ring;
        L.zero = L.csum = L.stcnt + digit_start_bytes(g, supers);
        L.done = L.csum + csum_bytes(g, supers);
        L.zero_bytes = csum_bytes(g, supers) + done_bytes;
    } else {
        L.zero = L.agg = L.ring;
        L.done = L.ring + count_word_bytes(g);
        L.csum = L.done + done_bytes;
        L.zero_bytes = count_word_bytes(g) + done_bytes + csum_bytes(g, supers);
        L.stcnt = L.ring + L.zero_bytes;
    }
    L.fin = L.ring;
    L.total = o;
    return L;
}

// HIP events recorded on the call's stream around each phase (RADSORT_F_TIMING).
enum Mark { kStart, kSetupEnd, kCountBegin, kRoundBegin, kRoundEnd, kFixupEnd, kFinBegin, kFinEnd };

struct Timer {
    static constexpr int kMax = 8 + 4 * RADSORT_MAX_ROUNDS;
    hipEvent_t ev[kMax];
    int tag[kMax], round[kMax];
    int count = 0;
    bool created = false, active = false, pending = false;

    void begin()
    {
        if (!created) {
            for (int i = 0; i < kMax; i++) (void)hipEventCreate(&ev[i]);
            created = true;
        }
        count = 0;
        active = true;
        pending = false;
    }
    void mark(Mark m, int r, hipStream_t s)
    {
        if (!active || count >= kMax) return;
        tag[count] = m;
        round[count] = r;
        (void)hipEventRecord(ev[count], s);
        count++;
    }
    void end()
    {
        if (active) pending = count > 0;
        active = false;
    }
    // waits for the last event and fills the timing fields of st
    void report(radsort_stats& st)
    {
        if (!pending) return;
        pending = false;
        if (hipEventSynchronize(ev[count - 1]) != hipSuccess) return;
        auto ms = [&](int a, int b) {
            float t = 0;
            (void)hipEventElapsedTime(&t, ev[a], ev[b]);
            return t;
        };
        st.timed = 1;
        st.setup_ms = st.fixup_ms = st.finalize_ms = 0;
        for (int r = 0; r < RADSORT_MAX_ROUNDS; r++) st.round_ms[r] = st.count_ms[r] = 0;
        st.total_ms = ms(0, count - 1);
        for (int i = 1; i < count; i++) {
            const float d = ms(i - 1, i);
            switch (tag[i]) {
            case kSetupEnd: st.setup_ms += d; break;
            case kRoundEnd: st.round_ms[round[i] % RADSORT_MAX_ROUNDS] += d; break;
            case kRoundBegin: st.count_ms[round[i] % RADSORT_MAX_ROUNDS] += d; break;
            case kCountBegin:
            case kFixupEnd: st.fixup_ms += d; break;
            case kFinEnd: st.finalize_ms += d; break;
            default: st.setup_ms += d; break;  // gaps before a finalize
            }
        }
    }
};

thread_local Timer g_timer;

void launch_fill(uint32_t* p, uint64_t count, uint32_t v, hipStream_t s)
{
    if (!count) return;
    uint32_t grid = (uint32_t)std::min<uint64_t>((count + 255) / 256, 4096);
    hipLaunchKernelGGL(k_fill_u32, dim3(grid), dim3(256), 0, s, p, count, v);
}

}  // namespace

struct radsort_state {
    Geo g;
    Layout L;
    uint8_t* ws = nullptr;
    bool own_ws = false;
    void* keys = nullptr;
    void* vals = nullptr;
    uint32_t rounds_done = 0;  // rounds since setup
    int cur = 0;               // which pi buffer holds pi
    uint64_t count = 0;        // elements in the dataset (fewer after truncate)
    bool truncated = false;
    bool is_setup = false;
    bool dynamic = false;      // launch forms that need no co-residency (shared GPU)
    bool shared = false;       // other work shares the GPU: no cooperative launch at all
    bool seq_draws = false;    // draws in the sequential pool order (RADSORT_F_SEQ_DRAWS)
    bool pack = false;         // the last round is packed (workspace laid out for it)
    int msd_shift = -1;        // >= 0: the rounds sort the digit at this shift (MSD split)
    bool debug_order = false;  // ordering-check builds: RADSORT_F_DEBUG_ORDER
    bool debug_plant = false;  // ... and RADSORT_F_DEBUG_PLANT: marks with a wrong tag
    uint32_t debug_seq = 0;    // the state's number, part of the round tags

    uint32_t* u32(uint64_t off) const { return (uint32_t*)(ws + off); }
    uint32_t* pi(int which) const { return u32(which ? L.pi1 : L.pi0); }
    PlanPtrs plan() const
    {
        return PlanPtrs{u32(L.S), u32(L.Pidx), u32(L.Plen), u32(L.f), u32(L.est)};
    }
    uint32_t* err() const { return u32(L.ctr) + g.nt; }
    // one-call sorts on the tile kernel: all rounds are planned ahead from one count of all
    // key positions (k_hist_plan; mode words 0 .. n_t - 1 of the counters), and tiles look
    // back over all earlier tiles, not over a counted super-tile's
    bool modes() const { return pack && g.tile && msd_shift < 0; }
    // a look-back word per (tile, digit) in the place of the ring and the digit starts
    // where they fit (st_log2), else a ring of them in the place of the ring; they are
    // zeroed per round
    bool chain_rows() const { return modes() && g.st_log2 == 0; }
    uint64_t zero_from() const { return chain_rows() ? L.stcnt : L.zero; }
    uint64_t zero_words() const { return (L.zero + L.zero_bytes - zero_from()) / 4; }
    // entries of pi: a packed round's extra blocks too
    uint32_t npx() const { return g.npi + (pack ? g.sigma : 0u); }
};

namespace {

// ---- launch helpers templated on key / payload widths --------------------------------

template <int KB> int launch_histograms(const void* keys, const Geo& g, uint32_t* hist,
                                        hipStream_t s)
{
    launch_fill(hist, (uint64_t)g.nt * g.sigma, 0, s);
    if (g.n == 0) return RADSORT_OK;
    // copies of the counts per workgroup: as many as fit in 32 KB, up to one per wave
    const uint32_t words = g.nt * g.sigma;
    const uint32_t copies = std::max<uint32_t>(1, std::min<uint32_t>(8, 8192 / words));
    uint32_t grid = (uint32_t)std::min<uint64_t>((g.n + 4095) / 4096, 2048);
    hipLaunchKernelGGL((k_histograms<KB, 512>), dim3(grid), dim3(512), 4 * copies * words, s,
                       (const typename UInt<KB>::T*)keys, g.n, g.bits, g.nt, copies, hist);
    return RADSORT_OK;
}

// Workgroups of `kern` that fit on the device at once (cached per device).
int resident_capacity(const void* kern, uint32_t threads)
{
    static std::mutex mu;
    static std::map<std::pair<int, const void*>, int> cache;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    std::lock_guard<std::mutex> lock(mu);
    auto it = cache.find({dev, kern});
    if (it != cache.end()) return it->second;
    int cus = 0, per = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kern, (int)threads, 0) != hipSuccess)
        return 0;
    cache[{dev, kern}] = cus * per;
    return cus * per;
}

// The round kernel is persistent: at most as many workgroups as fit at once, all
// resident (cooperative launch), each taking tiles in grid-stride order.
template <typename Args>
int launch_persistent(const void* kern, uint32_t tiles, uint32_t threads, Args& a, hipStream_t s)
{
    const int cap = resident_capacity(kern, threads);
    if (cap <= 0) return RADSORT_E_DEVICE;
    const uint32_t grid = std::min<uint32_t>(tiles, (uint32_t)cap);
    static const bool verbose = getenv("RADSORT_VERBOSE") != nullptr;
    if (verbose)
        fprintf(stderr, "radsort: persistent launch %u workgroups x %u threads for %u tiles\n",
                grid, threads, tiles);
    void* args[] = {(void*)&a};
    RS_HIP(hipLaunchCooperativeKernel(kern, dim3(grid), dim3(threads), args, 0, s));
    return RADSORT_OK;
}

// Digit starts of every super-tile of a round's input and the plan of round r from the
// digit totals (S[r], P[r+1], f[r+1], and est[r] for the out-of-place or packed round):
// one launch (k_supertile_counts).  Row `supers` of stcnt, past the input, ends with the
// digit totals.
template <int KB, bool OOP>
void launch_super_counts(const Geo& g, const typename UInt<KB>::T* Ak,
                         const typename UInt<KB>::T* Tk, const uint32_t* pi,
                         const uint32_t* blen, const uint32_t* f_in, uint32_t shift,
                         uint32_t* stcnt, uint32_t* csum, uint32_t* err, uint32_t* done_ctr,
                         uint32_t r, PlanPtrs p, hipStream_t s, bool packed)
{
    const uint32_t rows = (OOP ? g.oop_supers : g.supers) + 1;
    const uint32_t sts_log2 = OOP ? g.oop_st_log2 + (uint32_t)ilog2(g.oop_E)
                                  : g.st_log2 + (uint32_t)ilog2(g.E);
    const uint32_t sig = g.sigma, plan = OOP ? 2u : packed ? 3u : 1u;
    PlanPtrs pr{p.S + r * sig, p.Pidx + (r + 1) * sig, p.Plen + (r + 1) * sig, p.f + r + 1,
                p.est + r * sig};
    // 512 threads, four workgroups to a compute unit, or 1024 where there is at most one
    // super-tile per compute unit (2^24 pairs, 1042 rows: 30 against 38 us; 2^20 pairs,
    // 162 rows: 17.5 against 15.5 us)
    auto launch = [&](auto kern, uint32_t threads) {
        hipLaunchKernelGGL(kern, dim3(rows), dim3(threads), 0, s, Ak, Tk, pi, blen, f_in, g.n, shift,
                           g.bits, g.log2b, g.npi, sts_log2, stcnt, csum, err, done_ctr, plan, pr);
    };
    if (rows <= 256) launch(k_supertile_counts<KB, OOP, 1024>, 1024);
    else launch(k_supertile_counts<KB, OOP, 512>, 512);
}

// The claimed forms (no co-residency needed): one workgroup per tile, or for the
// claim loop at most as many workgroups as fit at once.  `lds`, for a claim loop beside other
// work: bytes of LDS that keep its workgroups to one per compute unit, those of other sorts
// included.  Two of them to a unit (the records of 12 bytes fit so since the loop needs 127
// registers) get in each other's way: 8 out-of-place sorts at once of 2^24 .. 2^24.5, 2^24.5 ..
// 2^26 and 2^26 .. 2^27 records (uint32 and uint64 keys, uint32 payload) sort 10.6, 13.0 and
// 15.5 G keys/s with what fits, 13.7, 14.8 and 16.6 with one per unit of each sort, 15.0, 16.1
// and 17.5 with one per unit of all.
template <typename Args>
int launch_dynamic(const void* kern, uint32_t tiles, uint32_t threads, Args& a, hipStream_t s,
                   bool loop, uint32_t lds = 0)
{
    uint32_t grid = tiles;
    if (loop) {
        const int cap = resident_capacity(kern, threads);
        if (cap <= 0) return RADSORT_E_DEVICE;
        grid = std::min<uint32_t>(tiles, lds ? std::min<uint32_t>((uint32_t)cap, device_cus())
                                             : (uint32_t)cap);
    }
    void* args[] = {(void*)&a};
    RS_HIP(hipLaunchKernel(kern, dim3(grid), dim3(threads), args, lds, s));
    return RADSORT_OK;
}

#ifndef RS_RADSORT_FORM
#define RS_RADSORT_FORM kPerTile
#endif
// seq: draws in the sequential pool order (pi as in the sequential algorithm);
// otherwise in (digit, block) order within a tile.  Digits of more than 8 bits
// always draw in the sequential order.  The out-of-place round draws nothing.
template <int KB, int VB, bool OOP>
int launch_round_t(const Geo& g, TileArgs<KB, VB>& a, hipStream_t s, bool dyn = false,
                   bool seq = true, bool shared = false)
{
    using N = TileCfg<KB, VB, false, OOP>;
    using Wd = TileCfg<KB, VB, true, OOP>;
    using NS = typename N::Shape;
    const uint32_t tiles = OOP ? (uint32_t)((g.n + g.oop_E - 1) / g.oop_E) : g.tiles;
    if (tiles == 0) return RADSORT_OK;
    if constexpr (!OOP) {
        if (g.tile && !seq) {
            using TL = TileShape<KB, VB, true>;
            using TS = TileShape<KB, VB, false>;
            auto pick = [&](auto chain) {
                constexpr int CH = decltype(chain)::value;
                if (g.tile_large)
                    return g.bits == 8
                               ? (const void*)&k_tile_round<KB, VB, 8, typename TL::Shape, CH>
                               : (const void*)&k_tile_round<KB, VB, 0, typename TL::Shape, CH>;
                return g.bits == 8 ? (const void*)&k_tile_round<KB, VB, 8, typename TS::Shape, CH>
                                   : (const void*)&k_tile_round<KB, VB, 0, typename TS::Shape, CH>;
            };
            const void* kern = a.rows     ? pick(std::integral_constant<int, kChainRows>{})
                               : a.ring64 ? pick(std::integral_constant<int, kChainRing>{})
                                          : pick(std::integral_constant<int, kChainNone>{});
            return launch_dynamic(kern, tiles, 64 * (g.tile_large ? TL::WAVES : TS::WAVES), a, s,
                                  false);
        }
    }
    if constexpr (!OOP && ((KB == 4 && VB <= 4) || (KB == 8 && VB == 0))) {
        if (g.large_tile) {  // 8-bit or narrower digits only (make_geo); a workgroup per tile
            using LS = typename LargeTile<KB>::Shape;
            constexpr int M = RS_RADSORT_FORM;
            const void* kern =
                seq ? (g.bits == 8 ? (const void*)&k_round<KB, VB, false, 8, 256, LS, M, true>
                                   : (const void*)&k_round<KB, VB, false, 0, 256, LS, M, true>)
                    : (g.bits == 8 ? (const void*)&k_round<KB, VB, false, 8, 256, LS, M, false>
                                   : (const void*)&k_round<KB, VB, false, 0, 256, LS, M, false>);
            return launch_dynamic(kern, tiles, 64 * LargeTile<KB>::WAVES, a, s, false);
        }
    }
    // shapes without register prefetch take a workgroup per tile (the persistent
    // form would hold the loop's state in registers the shape does not have)
    if (g.bits <= 8 && !N::PF) dyn = true;
    if (dyn) {
        // measured alone: one workgroup per tile for the Radsort round, the claim
        // loop for the out-of-place round
        constexpr int M = OOP ? kClaimLoop : RS_RADSORT_FORM;
        const uint32_t nt = 64 * N::WAVES;
        const void* kern;
        if (OOP || !seq)
            kern = g.bits == 8 ? (const void*)&k_round<KB, VB, OOP, 8, 256, NS, M, false>
                               : (const void*)&k_round<KB, VB, OOP, 0, 256, NS, M, false>;
        else
            kern = g.bits == 8 ? (const void*)&k_round<KB, VB, OOP, 8, 256, NS, M, true>
                               : (const void*)&k_round<KB, VB, OOP, 0, 256, NS, M, true>;
        // the loop's own LDS is 50 to 90 KB of a compute unit's 160: 32 more keep a second out
        if (g.bits <= 8)
            return launch_dynamic(kern, tiles, nt, a, s, OOP, OOP && shared ? 32u << 10 : 0u);
        return launch_dynamic(
            (const void*)&k_round<KB, VB, OOP, 0, 2048, typename Wd::Shape, M, !OOP>, tiles,
            64 * Wd::WAVES, a, s, OOP);
    }
    if constexpr (N::PF) {
        const void* kern;
        if (OOP || !seq)
            kern = g.bits == 8 ? (const void*)&k_round<KB, VB, OOP, 8, 256, NS, kPersistent, false>
                               : (const void*)&k_round<KB, VB, OOP, 0, 256, NS, kPersistent, false>;
        else
            kern = g.bits == 8 ? (const void*)&k_round<KB, VB, OOP, 8, 256, NS, kPersistent, true>
                               : (const void*)&k_round<KB, VB, OOP, 0, 256, NS, kPersistent, true>;
        if (g.bits <= 8) return launch_persistent(kern, tiles, 64 * N::WAVES, a, s);
    }
    return launch_persistent(
        (const void*)&k_round<KB, VB, OOP, 0, 2048, typename Wd::Shape, kPersistent, !OOP>, tiles,
        64 * Wd::WAVES, a, s);
}

template <int KB, int VB> struct Ops {
    using K = typename UInt<KB>::T;
    using V = typename Payload<VB>::T;

    static int setup(radsort_state* st, hipStream_t s)
    {
        const Geo& g = st->g;
        g_timer.mark(kStart, 0, s);
        // every round is planned later from its own digit counts
        const uint64_t from = st->modes() ? st->L.est : st->L.ctr;  // est, then the counters
        uint64_t work = std::max<uint64_t>(st->npx(), g.n & (g.b - 1));
        uint32_t grid = (uint32_t)std::min<uint64_t>((work + 255) / 256, 4096);
        hipLaunchKernelGGL((k_setup<KB, VB>), dim3(grid), dim3(256), 0, s, (K*)st->keys,
                           (V*)st->vals, (K*)(st->ws + st->L.Tk), (V*)(st->ws + st->L.Tv), g.n,
                           g.log2b, g.sigma, g.npi, st->npx(), st->pi(0), st->pi(1), st->u32(st->L.blen),
                           (uint64_t*)(st->ws + st->L.opened), st->u32(st->L.Pidx),
                           st->u32(st->L.Plen), st->u32(st->L.f), st->u32(st->zero_from()),
                           st->zero_words(), st->u32(from),
                           (uint32_t)((st->L.ctr - from) / 4 + g.nt + 8));
        if (st->modes()) {
            // 16384 keys to a workgroup, more where that makes over 2048 workgroups
            const uint64_t per = align_up(std::max<uint64_t>(16384, (g.n + 2047) / 2048), 8192);
            const dim3 grid((uint32_t)((g.n + per - 1) / per));
            auto* kern = g.bits == 8 ? k_hist_plan<KB, 8, 1024> : k_hist_plan<KB, 0, 1024>;
            hipLaunchKernelGGL(kern, grid, dim3(1024), 0, s, (const K*)st->keys, g.n, g.bits, g.nt,
                               g.log2b, (uint32_t)per, st->plan(), st->u32(st->L.ctr),
                               st->err() + 1);
        }
        g_timer.mark(kSetupEnd, 0, s);
        st->cur = 0;
        st->rounds_done = 0;
        st->count = g.n;
        st->truncated = false;
        st->is_setup = true;
        return RADSORT_OK;
    }

    // truncate (Alg. 8) between rounds; the rounds still to run plan themselves
    // from the shorter dataset
    static int truncate(radsort_state* st, uint64_t count, hipStream_t s)
    {
        const Geo& g = st->g;
        const uint32_t r = st->rounds_done;
        hipLaunchKernelGGL(k_truncate<256>, dim3(1), dim3(256), 4 * g.sigma, s,
                           st->u32(st->L.Pidx) + r * g.sigma, st->u32(st->L.Plen) + r * g.sigma,
                           st->u32(st->L.f) + r, st->u32(st->L.blen), g.sigma, g.log2b, count,
                           st->err());
        st->count = count;
        st->truncated = true;
        return RADSORT_OK;
    }

    // a new sort of the current contents: the state becomes the input of round 0
    static int restart(radsort_state* st, hipStream_t s)
    {
        const Geo& g = st->g;
        const uint32_t r = st->rounds_done;
        if (r) {
            hipLaunchKernelGGL(k_copy_u32, dim3((g.sigma + 255) / 256), dim3(256), 0, s,
                               st->u32(st->L.Pidx), st->u32(st->L.Pidx) + r * g.sigma, g.sigma);
            hipLaunchKernelGGL(k_copy_u32, dim3((g.sigma + 255) / 256), dim3(256), 0, s,
                               st->u32(st->L.Plen), st->u32(st->L.Plen) + r * g.sigma, g.sigma);
            hipLaunchKernelGGL(k_copy_u32, dim3(1), dim3(64), 0, s, st->u32(st->L.f),
                               st->u32(st->L.f) + r, 1u);
        }
        st->rounds_done = 0;
        return RADSORT_OK;
    }

    static int blocks(radsort_state* st, uint32_t* phys, uint32_t* len, hipStream_t s)
    {
        const Geo& g = st->g;
        const uint32_t m = g.npi - g.sigma;
        const uint32_t grid = std::max<uint32_t>(1, std::min<uint32_t>((m + 255) / 256, 4096));
        hipLaunchKernelGGL(k_block_table, dim3(grid), dim3(256), 0, s, st->pi(st->cur),
                           st->u32(st->L.blen), st->u32(st->L.f) + st->rounds_done, g.sigma,
                           g.npi, g.log2b, phys, len);
        return RADSORT_OK;
    }

    static int round(radsort_state* st, hipStream_t s)
    {
        const Geo& g = st->g;
        const uint32_t r = st->rounds_done;
        const uint32_t t = g.nt - 1 - r;  // key position of this round
        TileArgs<KB, VB> a{};
        (void)t;
        a.Ak = (K*)st->keys;
        a.Av = (V*)st->vals;
        a.Tk = (K*)(st->ws + st->L.Tk);
        a.Tv = (V*)(st->ws + st->L.Tv);
        a.pi_old = st->pi(st->cur);
        a.pi_new = st->pi(st->cur ^ 1);
        a.blen = st->u32(st->L.blen);
        a.f_in = st->u32(st->L.f) + r;
        a.S = st->u32(st->L.S) + r * g.sigma;
        a.opened = (uint64_t*)(st->ws + st->L.opened);
        a.agg = (uint32_t*)(st->ws + st->L.agg);
        a.done = (uint32_t*)(st->ws + st->L.done);
        a.err = st->err();
        a.tile_ctr = a.done + g.ring_w;  // zeroed with the ring
        a.shift = st->msd_shift >= 0 ? (uint32_t)st->msd_shift : g.bits * r;
        a.bits = g.bits;
        a.log2b = g.log2b;
        a.npi = g.npi;
        a.ring_log2 = g.ring_log2;
        a.st_log2 = g.st_log2;
        // the last round of a packed sort (plan_round): its buckets start at their final
        // offsets and it draws from sigma extra blocks first.  Which round that is, and
        // which ones are left out, the device decides where the tile kernel runs (modes).
        const bool modes = st->modes();
        const bool packed = st->pack && !modes && r + 1 == g.nt && st->msd_shift < 0;
        a.npi_x = packed || modes ? g.npi + g.sigma : g.npi;
        if (packed || modes) {
            a.pack_est = st->u32(st->L.est) + r * g.sigma;
            a.Xk = (K*)(st->ws + st->L.Xk);
            a.Xv = (V*)(st->ws + st->L.Xv);
        }
        if (modes) a.mode = st->u32(st->L.ctr) + r;
        if (st->chain_rows()) a.rows = (uint32_t*)(st->ws + st->L.stcnt);
        else if (modes) a.ring64 = (uint64_t*)(st->ws + st->L.agg);
#ifdef RS_TIMELINE
        a.tl = g.tiles <= g_tl_tiles ? g_tl : nullptr;
#endif
#ifdef RS_DEBUG_ORDER
        a.consumed = st->debug_order ? st->u32(st->L.consumed) : nullptr;
        a.tag = st->debug_seq << 8 | (r + 1);  // one per state and round
        a.tag_mark = st->debug_plant ? a.tag ^ 0x80u : a.tag;
#endif
        uint32_t* stcnt = (uint32_t*)(st->ws + st->L.stcnt);
        a.stbase = stcnt;
        a.stsum = st->u32(st->L.csum);
        // the ring is clear: setup or the previous round's fixup cleared it
        if (!modes) {
            g_timer.mark(kCountBegin, r, s);
            launch_super_counts<KB, false>(g, a.Ak, a.Tk, a.pi_old, a.blen, a.f_in, a.shift, stcnt,
                                           st->u32(st->L.csum), a.err, a.tile_ctr + 1, r,
                                           st->plan(), s, packed);
            g_timer.mark(kRoundBegin, r, s);
        }
        int rc = launch_round_t<KB, VB, false>(g, a, s, st->dynamic, st->seq_draws);
        if (rc) return rc;
        g_timer.mark(kRoundEnd, r, s);
        uint32_t grid = (uint32_t)std::min<uint64_t>((a.npi_x + 255) / 256, 4096);
        PlanPtrs p = st->plan();
        p = PlanPtrs{p.S + r * g.sigma, p.Pidx + r * g.sigma, p.Plen + r * g.sigma, p.f + r,
                     p.est + r * g.sigma};
        if (packed)
            hipLaunchKernelGGL(k_pack_fixup, dim3(grid), dim3(256), 0, s, st->pi(st->cur),
                               st->pi(st->cur ^ 1), p, g.sigma, g.npi);
        else
            hipLaunchKernelGGL(k_fixup, dim3(grid), dim3(256), 0, s, st->pi(st->cur),
                               st->pi(st->cur ^ 1), p, st->u32(st->L.blen), a.opened, g.sigma,
                               g.log2b, g.npi, a.npi_x, st->u32(st->zero_from()), st->zero_words(),
                               a.mode, r);
        g_timer.mark(kFixupEnd, r, s);
        st->cur ^= 1;
        st->rounds_done++;
        return RADSORT_OK;
    }

    static int finalize_seq(radsort_state* st, hipStream_t s)
    {
        const Geo& g = st->g;
        const uint32_t r = st->rounds_done;
        hipLaunchKernelGGL((k_finalize_seq<KB, VB, 1024>), dim3(1), dim3(1024), 0, s,
                           (K*)st->keys, (V*)st->vals, (K*)(st->ws + st->L.Tk),
                           (V*)(st->ws + st->L.Tv), st->pi(st->cur), st->u32(st->L.fin),
                           st->u32(st->L.Pidx) + r * g.sigma, st->u32(st->L.Plen) + r * g.sigma,
                           st->u32(st->L.f) + r, g.n, g.sigma, g.log2b, g.npi);
        return RADSORT_OK;
    }

    static int finalize(radsort_state* st, hipStream_t s)
    {
        const Geo& g = st->g;
        const uint32_t r = st->rounds_done;
        FinArgs<KB, VB> a{};
        a.Ak = (K*)st->keys;
        a.Av = (V*)st->vals;
        a.Tk = (K*)(st->ws + st->L.Tk);
        a.Tv = (V*)(st->ws + st->L.Tv);
        a.pi = st->pi(st->cur);
        a.Pidx = st->u32(st->L.Pidx) + r * g.sigma;
        a.Plen = st->u32(st->L.Plen) + r * g.sigma;
        a.f = st->u32(st->L.f) + r;
        a.n = g.n;
        a.sigma = g.sigma;
        a.log2b = g.log2b;
        a.npi = g.npi;
        a.npi_eq = g.npi;
        if (st->pack && r == g.nt && st->msd_shift < 0) {  // the last round was packed
            a.npi = g.npi + g.sigma;
            a.Xk = (K*)(st->ws + st->L.Xk);
            a.Xv = (V*)(st->ws + st->L.Xv);
            a.est = st->u32(st->L.est) + (r - 1) * g.sigma;
            a.S = st->u32(st->L.S) + (r - 1) * g.sigma;
            a.pack = st->u32(st->L.pack);
        }
        a.job = fin_job(a.npi);
        a.err = st->err();
        a.scratch = st->ws + st->L.fin;
        a.spare_pi = st->pi(st->cur ^ 1);
        a.spare_blen = st->u32(st->L.blen);
        g_timer.mark(kFinBegin, 0, s);
        int cap = 0;       // 0: the dynamic compaction
        uint32_t cus = 0;  // 0: F1 without a cooperative launch
        if (!st->dynamic) {
            const void* compact =
                (const void*)&k_fin_compact<KB, VB, fin_chunk<KB, VB>(), kCompactThreads>;
            cap = resident_capacity(compact, kCompactThreads);
            if (cap <= 0) return RADSORT_E_DEVICE;
        }
        if (!st->shared) {
            int dev = 0, n_cu = 0;
            RS_HIP(hipGetDevice(&dev));
            RS_HIP(hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev));
            cus = (uint32_t)n_cu;
        }
        const bool temps = a.pack ? g.fin_temps_pack : g.fin_temps;
        const int fr = finalize_parallel<KB, VB>(a, (uint32_t)cap, cus, temps, s);
        int rc = fr == -2 ? RADSORT_E_NOMEM : fr ? RADSORT_E_DEVICE : RADSORT_OK;
        g_timer.mark(kFinEnd, 0, s);
        return rc;
    }

    static int logical(radsort_state* st, void* ok, void* ov, hipStream_t s)
    {
        const Geo& g = st->g;
        const uint32_t r = st->rounds_done;
        const uint32_t grid = g.npi - g.sigma;
        hipLaunchKernelGGL((k_gather_logical<KB, VB, 256>), dim3(grid), dim3(256), 0, s,
                           (const K*)st->keys, (const V*)st->vals,
                           (const K*)(st->ws + st->L.Tk), (const V*)(st->ws + st->L.Tv),
                           st->pi(st->cur), st->u32(st->L.Pidx) + r * g.sigma,
                           st->u32(st->L.Plen) + r * g.sigma, st->u32(st->L.f) + r, g.sigma,
                           g.log2b, g.npi, (K*)ok, (V*)ov);
        return RADSORT_OK;
    }

    // Alg. 1 rounds, ping-ponging between the caller's arrays and the workspace
    static int oop_sort(void* keys, void* vals, const Geo& g, const Layout& L, uint8_t* ws,
                        bool dyn, bool shared, hipStream_t s)
    {
        // each round's element starts come from its own digit counts
        PlanPtrs p{(uint32_t*)(ws + L.S), (uint32_t*)(ws + L.Pidx), (uint32_t*)(ws + L.Plen),
                   (uint32_t*)(ws + L.f), (uint32_t*)(ws + L.est)};
        g_timer.mark(kStart, 0, s);
        uint32_t* ctr = (uint32_t*)(ws + L.ctr);
        launch_fill(ctr, g.nt + 8, 0, s);
        g_timer.mark(kSetupEnd, 0, s);
        K* bk[2] = {(K*)keys, (K*)(ws + L.alt_k)};
        V* bv[2] = {(V*)vals, (V*)(ws + L.alt_v)};
        for (uint32_t r = 0; r < g.nt; r++) {
            const uint32_t t = g.nt - 1 - r, from = r & 1;
            TileArgs<KB, VB> a{};
            a.Ak = bk[from];
            a.Av = bv[from];
            a.Tk = bk[from ^ 1];
            a.Tv = bv[from ^ 1];
            a.est = p.est + r * g.sigma;
            a.n = g.n;
            a.agg = (uint32_t*)(ws + L.agg);
            a.done = (uint32_t*)(ws + L.done);
            a.err = ctr + g.nt;
            a.tile_ctr = a.done + g.ring_w;  // zeroed with the ring
            a.shift = g.bits * (g.nt - 1 - t);
            a.bits = g.bits;
            a.log2b = g.log2b;
            a.ring_log2 = g.ring_log2;
            a.st_log2 = g.oop_st_log2;
            uint32_t* stcnt = (uint32_t*)(ws + L.stcnt);
            a.stbase = stcnt;
            a.stsum = (uint32_t*)(ws + L.csum);
            launch_fill((uint32_t*)(ws + L.zero), L.zero_bytes / 4, 0, s);
            g_timer.mark(kCountBegin, r, s);
            launch_super_counts<KB, true>(g, a.Ak, (const K*)nullptr, nullptr, nullptr, nullptr,
                                          a.shift, stcnt, (uint32_t*)(ws + L.csum), a.err,
                                          a.tile_ctr + 1, r, p, s, false);
            g_timer.mark(kRoundBegin, r, s);
            int rc = launch_round_t<KB, VB, true>(g, a, s, dyn, true, shared);
            if (rc) return rc;
            g_timer.mark(kRoundEnd, r, s);
        }
        g_timer.mark(kFinBegin, 0, s);
        if (g.nt & 1) {  // the result is in the workspace buffer: copy it back
            RS_HIP(hipMemcpyAsync(keys, bk[1], g.n * KB, hipMemcpyDeviceToDevice, s));
            if (VB) RS_HIP(hipMemcpyAsync(vals, bv[1], g.n * VB, hipMemcpyDeviceToDevice, s));
        }
        g_timer.mark(kFinEnd, 0, s);
        return RADSORT_OK;
    }
};

template <template <int, int> class F, typename... Args>
int dispatch(uint32_t kb, uint32_t vb, Args&&... args)
{
    if (kb == 4 && vb == 0) return F<4, 0>::run(args...);
    if (kb == 4 && vb == 4) return F<4, 4>::run(args...);
    if (kb == 4 && vb == 8) return F<4, 8>::run(args...);
    if (kb == 8 && vb == 0) return F<8, 0>::run(args...);
    if (kb == 8 && vb == 4) return F<8, 4>::run(args...);
    if (kb == 8 && vb == 8) return F<8, 8>::run(args...);
    return RADSORT_E_INVALID;
}

template <int KB, int VB> struct DoSetup {
    static int run(radsort_state* st, hipStream_t s) { return Ops<KB, VB>::setup(st, s); }
};
template <int KB, int VB> struct DoRound {
    static int run(radsort_state* st, hipStream_t s) { return Ops<KB, VB>::round(st, s); }
};
template <int KB, int VB> struct DoFinalize {
    static int run(radsort_state* st, hipStream_t s) { return Ops<KB, VB>::finalize(st, s); }
};
template <int KB, int VB> struct DoFinalizeSeq {
    static int run(radsort_state* st, hipStream_t s) { return Ops<KB, VB>::finalize_seq(st, s); }
};
template <int KB, int VB> struct DoTruncate {
    static int run(radsort_state* st, uint64_t count, hipStream_t s)
    {
        return Ops<KB, VB>::truncate(st, count, s);
    }
};
template <int KB, int VB> struct DoRestart {
    static int run(radsort_state* st, hipStream_t s) { return Ops<KB, VB>::restart(st, s); }
};
template <int KB, int VB> struct DoBlocks {
    static int run(radsort_state* st, uint32_t* phys, uint32_t* len, hipStream_t s)
    {
        return Ops<KB, VB>::blocks(st, phys, len, s);
    }
};
template <int KB, int VB> struct DoLogical {
    static int run(radsort_state* st, void* k, void* v, hipStream_t s)
    {
        return Ops<KB, VB>::logical(st, k, v, s);
    }
};
template <int KB, int VB> struct DoOop {
    static int run(void* k, void* v, const Geo& g, const Layout& L, uint8_t* ws, bool dyn,
                   bool shared, hipStream_t s)
    {
        return Ops<KB, VB>::oop_sort(k, v, g, L, ws, dyn, shared, s);
    }
};

// ---- out of place in the workspace (kernel_seg.hpp) -----------------------------------------

// Tile shapes of k_seg_round: 0: 2048 records, many workgroups of 4 waves to a compute unit
// (small lone arrays: tiles for all the compute units); 1: 8192 records (4096 of 12 bytes or
// more); 2: twice that.
template <int KB, int VB, int SHAPE> struct SegShape {
    static constexpr bool WIDE = KB + VB >= 12 || KB == 8;
    static constexpr int WAVES = SHAPE == 0 ? 4 : 8;
    static constexpr int ITEMS = SHAPE == 0 ? 8 : (WIDE ? 8 : 16) << (SHAPE - 1);
    using Shape = RoundShape<WAVES, ITEMS, false, true, 4>;
    static constexpr uint32_t E = 64 * WAVES * ITEMS;
};
uint32_t seg_tile(uint32_t kb, uint32_t vb, int shape)
{
    return shape == 0 ? 2048u : (kb + vb >= 12 || kb == 8 ? 4096u : 8192u) << (shape - 1);
}
constexpr uint64_t kSegLargeMin = 65536;  // average array of a batch for shape 2

// The tables of a group of at most `arrays` arrays and `tiles` tiles, at byte offsets from a
// 256-byte aligned base: what k_seg_clear zeroes first (hist .. rounds), then the rest.
struct SegTables {
    uint64_t hist, arrived, state, ctr, rounds, zero_bytes, arr, map, total;
};
SegTables seg_tables(uint32_t nt, uint64_t arrays, uint64_t tiles, uint64_t all_arrays,
                     uint64_t all_tiles)
{
    SegTables T{};
    uint64_t o = 0;
    auto take = [&](uint64_t bytes) {
        const uint64_t at = o;
        o = align_up(o + bytes, 256);
        return at;
    };
    T.hist = take(arrays * nt * 1024);
    T.arrived = take(arrays * 4);
    T.state = take(tiles * 1024);
    T.ctr = take(4 * nt);
    T.rounds = take(arrays * 4);
    T.zero_bytes = o;
    T.map = take(all_tiles * 4);
    T.arr = take(all_arrays * sizeof(SegArr));
    T.total = o;
    return T;
}

template <int KB, int VB>
SegArgs<KB, VB> seg_args(void* keys, void* vals, void* sk, void* sv, uint8_t* base,
                         const SegTables& T, uint32_t* err)
{
    SegArgs<KB, VB> a{};
    a.Ak = (typename UInt<KB>::T*)keys;
    a.Av = (typename Payload<VB>::T*)vals;
    a.Sk = (typename UInt<KB>::T*)sk;
    a.Sv = (typename Payload<VB>::T*)sv;
    a.arr = (const SegArr*)(base + T.arr);
    a.map = (uint32_t*)(base + T.map);
    a.hist = (uint32_t*)(base + T.hist);
    a.arrived = (uint32_t*)(base + T.arrived);
    a.rounds = (uint32_t*)(base + T.rounds);
    a.state = (uint32_t*)(base + T.state);
    a.ctr = (uint32_t*)(base + T.ctr);
    a.err = err;
    return a;
}

// The counting pass and the rounds of one group of `tiles` tiles.
template <int KB, int VB, int SHAPE>
void launch_seg_group(SegArgs<KB, VB> a, uint32_t tiles, hipStream_t s)
{
    using S = SegShape<KB, VB, SHAPE>;
    SegArgs<KB, 0> h{};
    h.Ak = a.Ak;
    h.arr = a.arr;
    h.map = a.map;
    h.a0 = a.a0;
    h.t0 = a.t0;
    h.na = a.na;
    h.group = a.group;
    h.hist = a.hist;
    h.arrived = a.arrived;
    h.rounds = a.rounds;
    h.err = a.err;
    hipLaunchKernelGGL((k_seg_hist<KB, 512>), dim3(tiles), dim3(512), 0, s, h, S::E);
    for (a.r = 0; a.r < (uint32_t)KB; a.r++)
        hipLaunchKernelGGL((k_seg_round<KB, VB, typename S::Shape>), dim3(tiles),
                           dim3(64 * S::WAVES), 0, s, a);
}

// The tile shape for one array and its tables, which `avail` bytes must hold (shape < 0: they
// do not).  Total of the out-of-place sort, shapes 0 / 1 / 2: uint32 pairs 42 / 53 / 77 us at
// 2^15, 47 / 55 / 78 at 2^16, - / 64 / 83 at 2^18, - / 103 / 112 at 2^21, - / 147 / 136 at 2^22, - / 394 /
// 348 at 2^24; uint64 + uint32 77 / 81 / 110 at 2^15, 88 / 87 / 114 at 2^16, 222 / 173 / 174 at 2^20,
// 344 / 244 / 207 at 2^21.
//
// Beside other work on the GPU the look-back over all tiles of a long array loses more than it
// saves: 8 sorts at once of 2^24.5 .. 2^26 records (uint32 and uint64 keys, uint32 payload)
// sort 11.6 G keys/s so and 16.1 by the rounds with counting passes (launch_dynamic); of 2^23
// .. 2^24 records 24.7 and 13.2, of 2^20 .. 2^23 26.4 and 8.0 G keys/s.
struct SegOne {
    int shape = -1;
    SegTables T{};
};
constexpr uint64_t kSegSharedEnd = 1ull << 24;  // a shared GPU: arrays below this
SegOne seg_one(const Geo& g, uint64_t avail, bool shared)
{
    SegOne one;
    if (g.n >= (shared ? kSegSharedEnd : 1ull << kSegValueBits)) return one;
    const bool wide = g.kb + g.vb >= 12 || g.kb == 8;
    int shape = g.n <= (wide ? 1u << 16 : 1u << 18) ? 0 : g.n < (wide ? 1u << 20 : 1u << 22) ? 1 : 2;
    for (; shape <= 2; shape++) {
        const uint32_t E = seg_tile(g.kb, g.vb, shape);
        const uint64_t tiles = (g.n + E - 1) / E;
        one.T = seg_tables(g.kb, 1, tiles, 1, tiles);
        if (one.T.total <= avail) {
            one.shape = shape;
            break;
        }
    }
    return one;
}

// One array sorted out of place: scratch planes sk, sv and tables at base.
template <int KB, int VB> struct DoSegOne {
    static int run(void* keys, void* vals, uint32_t n, void* sk, void* sv, uint8_t* base,
                   uint32_t* err, const SegOne& one, hipStream_t s)
    {
        const SegTables& T = one.T;
        const int shape = one.shape;
        SegArgs<KB, VB> a = seg_args<KB, VB>(keys, vals, sk, sv, base, T, err);
        a.na = 1;
        const uint32_t E = seg_tile(KB, VB, shape), tiles = (n + E - 1) / E;
        // the map is all zeros too, and ends where the array's entry begins
        const uint64_t words = T.arr / 4;
        const uint32_t grid = (uint32_t)std::min<uint64_t>((words + 255) / 256, 4096);
        hipLaunchKernelGGL(k_seg_clear, dim3(grid), dim3(256), 0, s, (uint32_t*)base, words,
                           (SegArr*)(base + T.arr), n, err);
        if (shape == 0) launch_seg_group<KB, VB, 0>(a, tiles, s);
        else if (shape == 1) launch_seg_group<KB, VB, 1>(a, tiles, s);
        else launch_seg_group<KB, VB, 2>(a, tiles, s);
        return RADSORT_OK;
    }
};

// Arrays of at most small_elems elements are sorted whole in LDS by k_sort_small, one
// workgroup each, with no workspace.  Two shapes: 4 waves and 2048 records, of which many
// share a compute unit, and 8 waves and the whole range.
uint32_t small_elems(uint32_t kb, uint32_t vb) { return (kb + vb >= 12) ? 4096u : 8192u; }
constexpr uint32_t kSmallShort = 2048;
constexpr uint32_t kSmallClasses = 4096;  // claims of a batch's longer arrays at most

// nseg arrays by offsets_dev, or one array of n1 elements (offsets_dev null), whose call's
// error word is err.  Where most arrays of a batch are longer ones, the large shape takes all
// of them, a workgroup per array: 3000 arrays, three of four of 6000 uint32 pairs and one of
// 1000, take 203 us so and 224 us with a launch of each shape.  Else each array falls to one
// of the two: a workgroup per array for the short ones, workgroups that claim classes of arrays
// for the longer ones (claim: a zeroed counter).  Up to kSmallClasses arrays a class is one
// array; at least one workgroup per eight classes, so that many short arrays are passed over
// quickly.  200 000 arrays of 24 to 31 uint32 pairs take 1.03 ms alone, 1.08 ms with one long
// array among them and 145.5 ms where the workgroups, no more than the long arrays, claimed the
// arrays one by one; 4096 arrays with 8 long ones 0.10 and 0.40 ms.  A lone array above 512
// elements takes the large shape: its lanes hold fewer items.  4096 arrays of 2^6 .. 2^13
// uint32 pairs: 151 us, and 177 us with the large shape alone.
template <int KB, int VB> struct DoSmall {
    static int run(void* keys, void* vals, const uint64_t* offsets_dev, uint32_t nseg, uint64_t n1,
                   uint32_t shorts, uint32_t longs, uint32_t* err, uint32_t* claim, hipStream_t s)
    {
        constexpr int ITEMS = KB + VB >= 12 ? 8 : 16;
        auto* k = (typename UInt<KB>::T*)keys;
        auto* v = (typename Payload<VB>::T*)vals;
        const bool one = offsets_dev == nullptr;
        const bool all = !one && longs >= shorts && longs > nseg / 2;  // the large shape alone
        if (one ? n1 <= 512 : shorts > 0 && !all)
            hipLaunchKernelGGL((k_sort_small<KB, VB, 4, 8, false>), dim3(nseg), dim3(256), 0, s, k, v,
                               offsets_dev, nseg, n1, 0u, err, (uint32_t*)nullptr, nseg);
        const uint32_t classes = std::min(nseg, kSmallClasses);
        const uint32_t grid = std::min(classes, std::max(std::min(longs, 1024u), classes / 8));
        if (one ? n1 > 512 : all)
            hipLaunchKernelGGL((k_sort_small<KB, VB, 8, ITEMS, false>), dim3(nseg), dim3(512), 0, s,
                               k, v, offsets_dev, nseg, n1, 0u, err, (uint32_t*)nullptr, nseg);
        else if (longs > 0)
            hipLaunchKernelGGL((k_sort_small<KB, VB, 8, ITEMS, true>), dim3(grid), dim3(512), 0, s, k,
                               v, offsets_dev, nseg, n1, kSmallShort, err, claim, classes);
        return RADSORT_OK;
    }
};

int check_args(void* keys, void* payload, uint64_t n, int payload_bytes)
{
    if (n > 0 && !keys) return RADSORT_E_INVALID;
    if (payload_bytes && n > 0 && !payload) return RADSORT_E_INVALID;
    if (!payload_bytes && payload) return RADSORT_E_INVALID;
    return RADSORT_OK;
}

int read_err(radsort_state* st, hipStream_t s, uint32_t* bits)
{
    uint32_t e = 0;
    RS_HIP(hipMemcpyAsync(&e, st->err(), 4, hipMemcpyDeviceToHost, s));
    RS_HIP(hipStreamSynchronize(s));
    if (bits) *bits = e;
    g_stats.error_bits = e;
    return (e & kErrOrder) ? RADSORT_E_ORDER : e ? RADSORT_E_TIMEOUT : RADSORT_OK;
}

}  // namespace

// ---- C ABI ---------------------------------------------------------------------------


// ---- many arrays at once ---------------------------------------------------------

// Arrays of at most small_elems() elements are sorted whole in LDS by k_sort_small (one
// workgroup each, no workspace).  Arrays up to wg_max_elems() share the scratch of up to
// kWgSlots workgroups in the workspace: those that fit half of it are sorted out of place
// there, group by group (kernel_seg.hpp), the others by k_radsort_wg, one workgroup per
// array, each with its part of the scratch as its T.  Larger ones run the Radsort steps in
// the dynamic launch form, spread over kSegLanes streams forked from the caller's
// stream, each lane with its own workspace.
constexpr uint32_t kSegLanes = 4;
struct SegChoice {
    uint32_t b, bits;
};

// block size and digit width for an array of n elements: the first class of the
// table whose max_log2n covers ceil(log2 n), else b = 2^ceil(log2 sqrt n) in
// [64, 2048] and 8-bit digits (b in Theta(sqrt n), Sec. 3)
SegChoice seg_choice(const radsort_seg_tuning* t, uint64_t n)
{
    const uint32_t lg = (uint32_t)ilog2(n);
    if (t)
        for (uint32_t c = 0; c < t->classes && c < RADSORT_SEG_CLASSES; c++)
            if (lg <= t->max_log2n[c] && t->block_elems[c]) return {t->block_elems[c], t->digit_bits[c]};
    const uint32_t b = std::min<uint32_t>(2048u, std::max<uint32_t>(64u, 1u << ((lg + 1) / 2)));
    return {b, 8u};
}

// The largest array the one-workgroup path takes: its limit, or lower when the
// tuning's first class with block_elems > 0 starts below it (arrays from that class
// on run on the lanes).  The host plan and the device list both use this bound.
uint64_t seg_wg_hi(const radsort_seg_tuning* t, uint64_t se)
{
    uint64_t hi = wg_max_elems();
    if (!t) return hi;
    for (uint32_t c = 0; c < t->classes && c < RADSORT_SEG_CLASSES; c++) {
        if (t->block_elems[c]) {
            const uint64_t below = c ? (1ull << std::min<uint32_t>(t->max_log2n[c - 1], 40)) : se;
            return std::max<uint64_t>(se, std::min<uint64_t>(hi, below));
        }
    }
    return hi;
}

// Arrays of the batch that are sorted out of place in groups (kernel_seg.hpp).
struct SegGroups {
    struct Group {
        uint32_t a0, na, t0, t1, id;  // first array, arrays, tiles [t0, t1), number (as k_seg_plan's)
    };
    std::vector<Group> groups;
    uint32_t count = 0, tiles = 0, G64 = 0;  // arrays, tiles, group size in 64 records
    uint64_t hi = 0;                         // arrays of at most hi elements
    int shape = 1;
    SegTables T{};
    uint64_t sk = 0, sv = 0;  // scratch planes, from the tables' base
};

// Groups for the arrays of sizes `n` (in order, all at most `top`) with `avail` bytes for scratch and tables:
// the largest scratch whose tables fit beside it.  Arrays larger than half the scratch take
// no part (a group is cut where the running size passes a multiple of the scratch less the
// largest array).
void plan_groups(SegGroups& S, const std::vector<uint32_t>& n, uint64_t top, uint32_t kb,
                 uint32_t vb, uint64_t avail)
{
    const uint64_t rec = kb + vb;
    for (uint64_t D64 = avail / (64 * rec); D64 >= 128;) {
        S.groups.clear();
        S.count = 0;
        uint64_t maxpad = 0, sum = 0;
        for (uint32_t x : n) {
            const uint64_t p = ((uint64_t)x + 63) / 64;
            if (p > D64 / 2) continue;
            maxpad = std::max(maxpad, p);
            sum += x;
            S.count++;
        }
        if (!S.count) return;
        S.hi = std::min(D64 / 2 * 64, top);
        S.shape = sum / S.count >= kSegLargeMin ? 2 : 1;
        const uint32_t E = seg_tile(kb, vb, S.shape);
        S.G64 = (uint32_t)(D64 - maxpad);
        uint64_t pos = 0, group = ~0ull;
        uint32_t arrays = 0, tiles = 0, amax = 0, tmax = 0;
        for (uint32_t x : n) {
            const uint64_t p = ((uint64_t)x + 63) / 64;
            if (p > D64 / 2) continue;
            if (pos / S.G64 != group) {
                group = pos / S.G64;
                S.groups.push_back({arrays, 0, tiles, tiles, (uint32_t)group});
            }
            arrays++;
            tiles += (x + E - 1) / E;
            pos += p;
            auto& g = S.groups.back();
            g.na++;
            g.t1 = tiles;
            amax = std::max(amax, g.na);
            tmax = std::max(tmax, g.t1 - g.t0);
        }
        S.tiles = tiles;
        S.T = seg_tables(kb, amax, tmax, S.count, S.tiles);
        S.sk = S.T.total;
        S.sv = align_up(S.sk + D64 * 64 * kb, 256);
        if (S.sv + D64 * 64 * vb <= avail) return;
        // the next smaller scratch, but none that the tables of all arrays and tiles alone
        // push out (the same for as long as the same arrays take part): 2 * 10^6 arrays of
        // 8193 keys, whose tables leave no room at all, are planned in 100 ms, not 600
        const uint64_t fixed = S.T.total - S.T.map;
        do D64 -= D64 / 16 + 1;
        while (D64 >= 128 && D64 / 2 >= maxpad && fixed + D64 * 64 * rec > avail);
    }
    S.count = 0;
    S.groups.clear();
}

struct SegPlan {
    SegGroups groups;
    std::vector<uint32_t> large;  // indices of the arrays that run the Radsort steps
    std::vector<uint32_t> lane;   // lane of each of them
    std::vector<SegChoice> choice;
    uint64_t wg_hi = 0;           // arrays of (small, wg_hi] elements take the one-workgroup path
    uint64_t lane_off[kSegLanes] = {}, lane_bytes[kSegLanes] = {};
    uint32_t wg_count = 0, wg_slots = 0;  // arrays of the one-workgroup path, workgroups
    uint64_t wg_off = 0, wg_slot_bytes = 0, wg_list_off = 0;
    uint64_t total = 0;
    uint32_t small_short = 0, small_long = 0;  // arrays of k_sort_small's two shapes
};

// Workgroups of the one-workgroup path (each with its own T); they never wait
// for each other, so they need not all be resident.
constexpr uint32_t kWgSlots = 256;

int make_seg_plan(SegPlan& P, const uint64_t* off, uint32_t nseg, int kb, int vb,
                  const radsort_seg_tuning* tuning, const radsort_opts* opts)
try {
    const uint32_t se = small_elems(kb, vb);
    P.wg_hi = seg_wg_hi(tuning, se);
    std::vector<std::pair<uint64_t, uint32_t>> big;
    std::vector<uint32_t> mid;
    for (uint32_t i = 0; i < nseg; i++) {
        if (off[i + 1] < off[i]) return RADSORT_E_INVALID;
        const uint64_t n = off[i + 1] - off[i];
        if (n <= 1) continue;
        if (n <= se) {
            (n > kSmallShort ? P.small_long : P.small_short)++;
            continue;
        }
        if (n <= P.wg_hi) {
            P.wg_count++;
            mid.push_back((uint32_t)n);
            continue;
        }
        big.push_back({n, i});
    }
    // largest first, each to the lane with the fewest elements so far
    std::sort(big.begin(), big.end(), [](auto& x, auto& y) { return x.first > y.first; });
    uint64_t load[kSegLanes] = {};
    for (auto& [n, i] : big) {
        uint32_t l = 0;
        for (uint32_t k = 1; k < kSegLanes; k++)
            if (load[k] < load[l]) l = k;
        load[l] += n;
        SegChoice c = seg_choice(tuning, n);
        radsort_opts o = opts ? *opts : radsort_opts{};
        o.block_elems = c.b;
        o.flags |= RADSORT_F_SHARED;  // the lanes run concurrently (run_one)
        Geo g;
        int rc = make_geo(g, n, kb, vb, (int)c.bits, &o);
        if (rc) return rc;
        P.lane_bytes[l] = std::max(P.lane_bytes[l], make_layout(g, false, true).total);
        P.large.push_back(i);
        P.lane.push_back(l);
        P.choice.push_back(c);
    }
    uint64_t o = 256;  // error words and the one-workgroup path's claim counter
    for (uint32_t l = 0; l < kSegLanes; l++) {
        P.lane_off[l] = o;
        o = align_up(o + P.lane_bytes[l], 256);
    }
    if (P.wg_count) {
        P.wg_slots = std::min(P.wg_count, kWgSlots);
        P.wg_slot_bytes = wg_slot_bytes(kb, vb);
        P.wg_list_off = o;
        o = align_up(o + 4ull * P.wg_count, 256);
        P.wg_off = o;
        o += (uint64_t)P.wg_slots * P.wg_slot_bytes;
        plan_groups(P.groups, mid, P.wg_hi, kb, vb, (uint64_t)P.wg_slots * P.wg_slot_bytes);
    }
    P.total = o;
    return RADSORT_OK;
} catch (const std::bad_alloc&) {  // no exception leaves a C entry point
    return RADSORT_E_NOMEM;
}

struct LaneStreams {
    hipStream_t s[kSegLanes];
    hipEvent_t fork, join[kSegLanes];
};

// streams and events of the lanes, one set per device, kept until the process ends
int lane_streams(LaneStreams** out)
{
    static std::mutex mu;
    static std::map<int, LaneStreams*> sets;
    int dev = 0;
    RS_HIP(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lock(mu);
    auto it = sets.find(dev);
    if (it != sets.end()) {
        *out = it->second;
        return RADSORT_OK;
    }
    LaneStreams* L = new (std::nothrow) LaneStreams();
    if (!L) return RADSORT_E_NOMEM;
    for (uint32_t l = 0; l < kSegLanes; l++) {
        RS_HIP(hipStreamCreateWithFlags(&L->s[l], hipStreamNonBlocking));
        RS_HIP(hipEventCreateWithFlags(&L->join[l], hipEventDisableTiming));
    }
    RS_HIP(hipEventCreateWithFlags(&L->fork, hipEventDisableTiming));
    sets[dev] = L;
    *out = L;
    return RADSORT_OK;
}

// The arrays of the middle path: those that fit go through the groups, the others, one
// after the other on the same memory, through the one-workgroup kernel.
template <int KB, int VB> struct DoWg {
    static int run(void* keys, void* vals, const uint64_t* offsets_dev, uint32_t nseg,
                   const SegPlan& P, uint8_t* ws, uint32_t* claim, uint32_t* err, hipStream_t s)
    {
        using C = WgCfg<KB, VB>;
        const SegGroups& S = P.groups;
        uint8_t* const base = ws + P.wg_off;
        uint64_t lo = small_elems(KB, VB);
        if (S.count) {
            const uint32_t E = seg_tile(KB, VB, S.shape);
            SegArr* arr = (SegArr*)(base + S.T.arr);
            uint32_t* map = (uint32_t*)(base + S.T.map);
            hipLaunchKernelGGL(k_seg_plan<1024>, dim3(1), dim3(1024), 0, s, offsets_dev, nseg, lo,
                               S.hi, S.G64, E, arr, S.count, map, S.tiles);
            hipLaunchKernelGGL(k_seg_map, dim3(S.count), dim3(64), 0, s, (const SegArr*)arr, E,
                               S.tiles, map);
            SegArgs<KB, VB> a =
                seg_args<KB, VB>(keys, vals, base + S.sk, base + S.sv, base, S.T, err);
            for (const auto& g : S.groups) {
                const uint64_t words = S.T.zero_bytes / 4;
                const uint32_t grid = (uint32_t)std::min<uint64_t>((words + 255) / 256, 4096);
                hipLaunchKernelGGL(k_seg_clear, dim3(grid), dim3(256), 0, s, (uint32_t*)base, words,
                                   (SegArr*)nullptr, 0u, err);
                a.a0 = g.a0;
                a.na = g.na;
                a.t0 = g.t0;
                a.group = g.id;
                if (S.shape == 1) launch_seg_group<KB, VB, 1>(a, g.t1 - g.t0, s);
                else launch_seg_group<KB, VB, 2>(a, g.t1 - g.t0, s);
            }
            lo = std::max(lo, S.hi);
        }
        const uint32_t rest = P.wg_count - S.count;
        if (!rest) return RADSORT_OK;
        uint32_t* list = (uint32_t*)(ws + P.wg_list_off);
        hipLaunchKernelGGL(k_wg_list, dim3(1), dim3(1024), 0, s, offsets_dev, nseg, lo, P.wg_hi,
                           list, rest);
        hipLaunchKernelGGL((k_radsort_wg<KB, VB>), dim3(std::min(rest, P.wg_slots)), dim3(C::NT), 0,
                           s, (typename UInt<KB>::T*)keys, (typename Payload<VB>::T*)vals,
                           offsets_dev, nseg, (const uint32_t*)list, rest, claim, base,
                           P.wg_slot_bytes, err);
        return RADSORT_OK;
    }
};

__global__ void k_or_error(const uint32_t* src, uint32_t* dst)
{
    if (threadIdx.x == 0 && *src) atomicOr(dst, *src);
}

// pack: the state's last round is packed (one-call sorts), its workspace laid out
// for that (make_layout)
static int state_create(radsort_state** out, void* keys, void* payload, uint64_t n, int key_bytes,
                 int payload_bytes, int digit_bits, const radsort_opts* opts, bool pack);

// the Radsort steps of one array on stream s, in the dynamic launch form; its
// device error bits are ORed into *errs
int run_one(void* keys, void* vals, uint64_t n, int kb, int vb, SegChoice c, uint8_t* ws,
            uint64_t ws_bytes, uint32_t* errs, hipStream_t s)
{
    radsort_opts o{};
    o.block_elems = c.b;
    o.flags = RADSORT_F_SHARED;  // sized as the plan sized it
    o.workspace = ws;
    o.workspace_bytes = ws_bytes;
    radsort_state* st = nullptr;
    int rc = state_create(&st, keys, vals, n, kb, vb, (int)c.bits, &o, true);
    if (rc) return rc;
    st->dynamic = true;
    st->shared = true;  // the lanes run concurrently: no cooperative launch
    rc = radsort_state_setup(st, s);
    for (uint32_t r = 0; !rc && r < st->g.nt; r++) rc = radsort_state_round(st, s);
    if (!rc) rc = radsort_state_finalize(st, s);
    if (!rc) hipLaunchKernelGGL(k_or_error, dim3(1), dim3(64), 0, s, st->err(), errs);
    radsort_state_destroy(st);
    return rc;
}

// One-call sorts of arrays that one workgroup sorts on chip.  The result does not depend on
// the digits or the blocks.  A caller workspace is checked as for the other paths, and its
// error word cleared; without one nothing is allocated, and the call waits for the stream
// as it does where a workspace has to be freed.
static bool sort_is_small(const Geo& g, const radsort_opts* opts)
{
#ifdef RS_DEBUG_ORDER
    if (opts && (opts->flags & RADSORT_F_DEBUG_ORDER)) return false;
#endif
    (void)opts;
    return g.n <= small_elems(g.kb, g.vb);
}
// A one-call sort whose array fits its own workspace once more (T and the extra blocks hold
// 3 sigma b records) runs out of place there: 2 launches and one per key byte (6 of 4-byte
// keys) instead of some twenty.
static SegOne sort_in_workspace_plan(const radsort_state* st)
{
    const Geo& g = st->g;
    const uint64_t room = st->L.total - st->L.Tk, records = g.n * (g.kb + g.vb) + 256;
    if (st->debug_order || records > room) return SegOne{};
    return seg_one(g, room - records, st->shared);
}
static int sort_in_workspace(radsort_state* st, const SegOne& one, hipStream_t s)
{
    const Geo& g = st->g;
    uint8_t* const base = st->ws + st->L.Tk;
    g_timer.mark(kStart, 0, s);
    int rc = dispatch<DoSegOne>(g.kb, g.vb, st->keys, st->vals, (uint32_t)g.n,
                                (void*)(base + one.T.total),
                                (void*)(base + align_up(one.T.total + g.n * g.kb, 256)), base,
                                st->err(), one, s);
    g_timer.mark(kRoundEnd, 0, s);
    if (!rc) RS_HIP(hipGetLastError());
    return rc;
}
static int sort_small(void* keys, void* payload, const Geo& g, const Layout& L,
                      const radsort_opts* opts, hipStream_t s)
{
    uint32_t* err = nullptr;
    if (opts && opts->workspace) {
        if (opts->workspace_bytes < L.total) return RADSORT_E_NOMEM;
        err = (uint32_t*)((uint8_t*)opts->workspace + L.ctr) + g.nt;
    }
    const bool timing = opts && (opts->flags & RADSORT_F_TIMING);
    if (timing) g_timer.begin();
    g_timer.mark(kStart, 0, s);
    int rc = dispatch<DoSmall>(g.kb, g.vb, keys, payload, (const uint64_t*)nullptr, 1u, g.n, 0u, 0u, err,
                               (uint32_t*)nullptr, s);
    g_timer.mark(kRoundEnd, 0, s);
    g_timer.end();
    g_stats.timed = 0;
    g_stats.workspace_bytes = L.total;
    g_stats.input_bytes = g.n * (uint64_t)(g.kb + g.vb);
    g_stats.rounds = g.nt;
    if (!rc) RS_HIP(hipGetLastError());
    if (!rc && (!err || (opts->flags & RADSORT_F_CHECK))) {
        RS_HIP(hipStreamSynchronize(s));
        g_stats.error_bits = 0;
    }
    return rc;
}

static int state_create(radsort_state** out, void* keys, void* payload, uint64_t n, int key_bytes,
                 int payload_bytes, int digit_bits, const radsort_opts* opts, bool pack)
{
    if (!out) return RADSORT_E_INVALID;
    *out = nullptr;
    int rc = check_args(keys, payload, n, payload_bytes);
    if (rc) return rc;
    Geo g;
    rc = make_geo(g, n, key_bytes, payload_bytes, digit_bits, opts);
    if (rc) return rc;
    radsort_state* st = new (std::nothrow) radsort_state();
    if (!st) return RADSORT_E_NOMEM;
    st->g = g;
    st->pack = pack;
    st->L = make_layout(g, false, pack);
    st->keys = keys;
    st->vals = payload;
    st->count = n;
    st->seq_draws = opts && (opts->flags & RADSORT_F_SEQ_DRAWS);
#ifdef RS_DEBUG_ORDER
    static std::atomic<uint32_t> debug_states{0};
    st->debug_order = opts && (opts->flags & RADSORT_F_DEBUG_ORDER);
    st->debug_plant = st->debug_order && (opts->flags & RADSORT_F_DEBUG_PLANT);
    st->debug_seq = (debug_states.fetch_add(1) + 1) & 0xFFFFFFu;
#endif
    if (opts && opts->workspace) {
        if (opts->workspace_bytes < st->L.total) {
            delete st;
            return RADSORT_E_NOMEM;
        }
        st->ws = (uint8_t*)opts->workspace;
    } else {
        hipError_t e = hipMalloc((void**)&st->ws, st->L.total);
        if (e != hipSuccess) {
            g_last_hip = e;
            delete st;
            return RADSORT_E_NOMEM;
        }
        st->own_ws = true;
    }
    *out = st;
    return RADSORT_OK;
}

extern "C" {

int radsort_state_create(radsort_state** out, void* keys, void* payload, uint64_t n,
                         int key_bytes, int payload_bytes, int digit_bits,
                         const radsort_opts* opts)
{
    return state_create(out, keys, payload, n, key_bytes, payload_bytes, digit_bits, opts, false);
}

int radsort_state_setup(radsort_state* st, void* stream)
{
    if (!st) return RADSORT_E_INVALID;
    int rc = dispatch<DoSetup>(st->g.kb, st->g.vb, st, (hipStream_t)stream);
    if (rc) return rc;
    RS_HIP(hipGetLastError());
    return RADSORT_OK;
}

int radsort_state_round(radsort_state* st, void* stream)
{
    if (!st || !st->is_setup || st->rounds_done >= st->g.nt) return RADSORT_E_INVALID;
    int rc = dispatch<DoRound>(st->g.kb, st->g.vb, st, (hipStream_t)stream);
    if (rc) return rc;
    RS_HIP(hipGetLastError());
    return RADSORT_OK;
}

int radsort_state_finalize(radsort_state* st, void* stream)
{
    if (!st || !st->is_setup) return RADSORT_E_INVALID;
    int rc = dispatch<DoFinalize>(st->g.kb, st->g.vb, st, (hipStream_t)stream);
    if (rc) return rc;
    RS_HIP(hipGetLastError());
    st->is_setup = false;
    return RADSORT_OK;
}

int radsort_state_finalize_sequential(radsort_state* st, void* stream)
{
    if (!st || !st->is_setup) return RADSORT_E_INVALID;
    if (st->truncated) return RADSORT_E_UNSUPPORTED;
    int rc = dispatch<DoFinalizeSeq>(st->g.kb, st->g.vb, st, (hipStream_t)stream);
    if (rc) return rc;
    RS_HIP(hipGetLastError());
    st->is_setup = false;
    return RADSORT_OK;
}

int radsort_state_read(radsort_state* st, uint32_t* pi, uint32_t* P_idx, uint32_t* P_len,
                       uint32_t* f, void* stream)
{
    if (!st) return RADSORT_E_INVALID;
    hipStream_t s = (hipStream_t)stream;
    const Geo& g = st->g;
    const uint32_t r = st->rounds_done;
    if (pi) RS_HIP(hipMemcpyAsync(pi, st->pi(st->cur), 4ull * g.npi, hipMemcpyDeviceToHost, s));
    if (P_idx)
        RS_HIP(hipMemcpyAsync(P_idx, st->u32(st->L.Pidx) + r * g.sigma, 4ull * g.sigma,
                              hipMemcpyDeviceToHost, s));
    if (P_len)
        RS_HIP(hipMemcpyAsync(P_len, st->u32(st->L.Plen) + r * g.sigma, 4ull * g.sigma,
                              hipMemcpyDeviceToHost, s));
    if (f) RS_HIP(hipMemcpyAsync(f, st->u32(st->L.f) + r, 4, hipMemcpyDeviceToHost, s));
    return read_err(st, s, nullptr);
}

int radsort_state_truncate(radsort_state* st, uint64_t count, void* stream)
{
    if (!st || !st->is_setup || count > st->count) return RADSORT_E_INVALID;
    int rc = dispatch<DoTruncate>(st->g.kb, st->g.vb, st, count, (hipStream_t)stream);
    if (rc) return rc;
    RS_HIP(hipGetLastError());
    return RADSORT_OK;
}

int radsort_state_restart(radsort_state* st, void* stream)
{
    if (!st || !st->is_setup) return RADSORT_E_INVALID;
    int rc = dispatch<DoRestart>(st->g.kb, st->g.vb, st, (hipStream_t)stream);
    if (rc) return rc;
    RS_HIP(hipGetLastError());
    return RADSORT_OK;
}

int radsort_state_blocks(radsort_state* st, uint32_t* phys, uint32_t* len, void* stream)
{
    if (!st || !st->is_setup || (!phys && !len)) return RADSORT_E_INVALID;
    int rc = dispatch<DoBlocks>(st->g.kb, st->g.vb, st, phys, len, (hipStream_t)stream);
    if (rc) return rc;
    RS_HIP(hipGetLastError());
    return RADSORT_OK;
}

int radsort_state_planes(const radsort_state* st, void** t_keys, void** t_payload,
                         uint32_t* block_elems)
{
    if (!st) return RADSORT_E_INVALID;
    if (t_keys) *t_keys = st->ws + st->L.Tk;
    if (t_payload) *t_payload = st->g.vb ? (void*)(st->ws + st->L.Tv) : nullptr;
    if (block_elems) *block_elems = st->g.b;
    return RADSORT_OK;
}

int radsort_state_count(const radsort_state* st, uint64_t* count)
{
    if (!st || !count) return RADSORT_E_INVALID;
    *count = st->count;
    return RADSORT_OK;
}

int radsort_state_logical(radsort_state* st, void* keys_out, void* payload_out, void* stream)
{
    if (!st || !st->is_setup) return RADSORT_E_INVALID;
    if ((st->count && !keys_out) || (st->g.vb && st->count && !payload_out))
        return RADSORT_E_INVALID;
    int rc = dispatch<DoLogical>(st->g.kb, st->g.vb, st, keys_out, payload_out,
                                 (hipStream_t)stream);
    if (rc) return rc;
    RS_HIP(hipGetLastError());
    return RADSORT_OK;
}

int radsort_state_dims(const radsort_state* st, uint32_t* npi, uint32_t* sigma, uint32_t* nt)
{
    if (!st) return RADSORT_E_INVALID;
    if (npi) *npi = st->g.npi;
    if (sigma) *sigma = st->g.sigma;
    if (nt) *nt = st->g.nt;
    return RADSORT_OK;
}

int radsort_state_destroy(radsort_state* st)
{
    if (!st) return RADSORT_OK;
    if (st->own_ws && st->ws) (void)hipFree(st->ws);
    delete st;
    return RADSORT_OK;
}

uint64_t radsort_workspace_bytes(uint64_t n, int key_bytes, int payload_bytes, int digit_bits,
                                 const radsort_opts* opts)
{
    Geo g;
    if (make_geo(g, n, key_bytes, payload_bytes, digit_bits, opts)) return 0;
    return make_layout(g, false, true).total;
}

uint64_t radsort_oop_workspace_bytes(uint64_t n, int key_bytes, int payload_bytes,
                                     int digit_bits, const radsort_opts* opts)
{
    Geo g;
    if (make_geo(g, n, key_bytes, payload_bytes, digit_bits, opts)) return 0;
    return make_layout(g, true).total;
}

int radsort_workspace_error(const void* workspace, uint64_t n, int key_bytes, int payload_bytes,
                            int digit_bits, const radsort_opts* opts, int out_of_place,
                            uint32_t* error_bits, void* stream)
{
    if (error_bits) *error_bits = 0;
    if (!workspace || !opts) return RADSORT_E_INVALID;
    Geo g;
    int rc = make_geo(g, n, key_bytes, payload_bytes, digit_bits, opts);
    if (rc) return rc;
    if (n <= 1) return RADSORT_OK;  // such a call runs nothing
    // the error word lies among the small arrays at the front of every layout
    const Layout L = make_layout(g, out_of_place != 0);
    if (opts->workspace_bytes < L.ctr + 4ull * (g.nt + 1)) return RADSORT_E_NOMEM;
    hipStream_t s = (hipStream_t)stream;
    uint32_t e = 0;
    RS_HIP(hipMemcpyAsync(&e, (const uint8_t*)workspace + L.ctr + 4ull * g.nt, 4,
                          hipMemcpyDeviceToHost, s));
    RS_HIP(hipStreamSynchronize(s));
    if (error_bits) *error_bits = e;
    return (e & kErrOrder) ? RADSORT_E_ORDER : e ? RADSORT_E_TIMEOUT : RADSORT_OK;
}

int radsort_sort_pairs(void* keys, void* payload, uint64_t n, int key_bytes, int payload_bytes,
                       int digit_bits, const radsort_opts* opts, void* stream)
{
    int rc = check_args(keys, payload, n, payload_bytes);
    if (rc) return rc;
    Geo g;
    rc = make_geo(g, n, key_bytes, payload_bytes, digit_bits, opts);
    if (rc) return rc;
    if (n <= 1) return RADSORT_OK;
    if (sort_is_small(g, opts)) return sort_small(keys, payload, g, make_layout(g, false, true), opts, (hipStream_t)stream);
    radsort_state* st = nullptr;
    rc = state_create(&st, keys, payload, n, key_bytes, payload_bytes, digit_bits, opts, true);
    if (rc) return rc;
    // The launch form without co-residency (one workgroup per tile) is also the
    // faster one alone for blocks of up to 1024 elements (no cooperative launch per
    // round, which costs most at small n); with larger blocks the persistent form,
    // whose workgroups overlap one tile's loads with the previous tile, is faster.
    st->dynamic = (opts && (opts->flags & RADSORT_F_SHARED)) || g.b <= 1024;
    st->shared = opts && (opts->flags & RADSORT_F_SHARED);
    hipStream_t s = (hipStream_t)stream;
    const bool timing = opts && (opts->flags & RADSORT_F_TIMING);
    if (timing) g_timer.begin();
    const SegOne one = sort_in_workspace_plan(st);
    if (one.shape >= 0) {
        rc = sort_in_workspace(st, one, s);
    } else {
        rc = radsort_state_setup(st, s);
        for (uint32_t r = 0; !rc && r < st->g.nt; r++) rc = radsort_state_round(st, s);
        if (!rc) rc = radsort_state_finalize(st, s);
    }
    g_timer.end();
    g_stats.timed = 0;
    g_stats.workspace_bytes = st->L.total;
    g_stats.input_bytes = n * (uint64_t)(key_bytes + payload_bytes);
    g_stats.rounds = st->g.nt;
    const bool check = opts && (opts->flags & RADSORT_F_CHECK);
    if (!rc && (check || st->own_ws)) rc = read_err(st, s, nullptr);
    radsort_state_destroy(st);  // a library-owned workspace is freed after read_err's wait
    return rc;
}

int radsort_sort(void* keys, uint64_t n, int key_bytes, int digit_bits, void* stream)
{
    return radsort_sort_pairs(keys, nullptr, n, key_bytes, 0, digit_bits, nullptr, stream);
}

int radsort_oop_sort_pairs(void* keys, void* payload, uint64_t n, int key_bytes,
                           int payload_bytes, int digit_bits, const radsort_opts* opts,
                           void* stream)
{
    int rc = check_args(keys, payload, n, payload_bytes);
    if (rc) return rc;
    Geo g;
    rc = make_geo(g, n, key_bytes, payload_bytes, digit_bits, opts);
    if (rc) return rc;
    if (n <= 1) return RADSORT_OK;
    Layout L = make_layout(g, true);
    hipStream_t s = (hipStream_t)stream;
    if (sort_is_small(g, opts)) return sort_small(keys, payload, g, L, opts, s);
    uint8_t* ws = nullptr;
    bool own = false;
    if (opts && opts->workspace) {
        if (opts->workspace_bytes < L.total) return RADSORT_E_NOMEM;
        ws = (uint8_t*)opts->workspace;
    } else {
        hipError_t e = hipMalloc((void**)&ws, L.total);
        if (e != hipSuccess) {
            g_last_hip = e;
            return RADSORT_E_NOMEM;
        }
        own = true;
    }
    const bool timing = opts && (opts->flags & RADSORT_F_TIMING);
    if (timing) g_timer.begin();
    // the out-of-place round runs faster in the form without co-residency (one
    // workgroup per tile) at every size and block tried, so it always takes it
    const bool dyn = true;
    const bool shared = opts && (opts->flags & RADSORT_F_SHARED);
    const SegOne one = seg_one(g, L.total - L.ring, shared);
    if (one.shape >= 0) {
        g_timer.mark(kStart, 0, s);
        rc = dispatch<DoSegOne>(g.kb, g.vb, keys, payload, (uint32_t)n, (void*)(ws + L.alt_k),
                                (void*)(ws + L.alt_v), ws + L.ring, (uint32_t*)(ws + L.ctr) + g.nt,
                                one, s);
        g_timer.mark(kRoundEnd, 0, s);
    } else {
        rc = dispatch<DoOop>(g.kb, g.vb, keys, payload, g, L, ws, dyn, shared, s);
    }
    g_timer.end();
    g_stats.timed = 0;
    if (!rc) {
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) {
            g_last_hip = e;
            rc = RADSORT_E_DEVICE;
        }
    }
    g_stats.workspace_bytes = L.total;
    g_stats.input_bytes = n * (uint64_t)(key_bytes + payload_bytes);
    g_stats.rounds = g.nt;
    const bool check = opts && (opts->flags & RADSORT_F_CHECK);
    if (!rc && (check || own)) {
        uint32_t e = 0;
        hipError_t he = hipMemcpyAsync(&e, ws + L.ctr + 4ull * g.nt, 4, hipMemcpyDeviceToHost, s);
        if (he == hipSuccess) he = hipStreamSynchronize(s);
        if (he != hipSuccess) {
            g_last_hip = he;
            rc = RADSORT_E_DEVICE;
        } else if (e) {
            rc = RADSORT_E_TIMEOUT;
        }
        g_stats.error_bits = e;
    }
    if (own) {
        (void)hipStreamSynchronize(s);
        (void)hipFree(ws);
    }
    return rc;
}

int radsort_histograms(const void* keys, uint64_t n, int key_bytes, int digit_bits,
                       uint32_t* counts, void* stream)
{
    if (!counts || (n && !keys)) return RADSORT_E_INVALID;
    Geo g;
    int rc = make_geo(g, n, key_bytes, 0, digit_bits, nullptr);
    if (rc) return rc;
    hipStream_t s = (hipStream_t)stream;
    rc = key_bytes == 4 ? launch_histograms<4>(keys, g, counts, s)
                        : launch_histograms<8>(keys, g, counts, s);
    if (rc) return rc;
    RS_HIP(hipGetLastError());
    return RADSORT_OK;
}

int radsort_last_stats(radsort_stats* out)
{
    if (!out) return RADSORT_E_INVALID;
    g_timer.report(g_stats);
    *out = g_stats;
    return RADSORT_OK;
}

int radsort_copy(void* dst, const void* src, uint64_t bytes, void* stream)
{
    if (bytes && (!dst || !src)) return RADSORT_E_INVALID;
    if (((uintptr_t)dst | (uintptr_t)src) & 15) return RADSORT_E_INVALID;
    if (!bytes) return RADSORT_OK;
    const uint64_t words = bytes / 16;
    const uint32_t tail = (uint32_t)(bytes % 16);
    int dev = 0, cus = 0;
    RS_HIP(hipGetDevice(&dev));
    RS_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    // one workgroup of 256 threads per CU (fewer when there is less to copy): with
    // 4 words in flight per thread this is the fastest of the shapes measured on
    // MI355X (5.7 TB/s for 2 GiB; 8 workgroups per CU: 4.7 TB/s, 2: 5.5 TB/s)
    const uint64_t want = (words + 4 * 256 - 1) / (4 * 256);
    const uint32_t grid = (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(want, (uint64_t)cus));
    hipLaunchKernelGGL(k_stream_copy, dim3(grid), dim3(256), 0, (hipStream_t)stream,
                       (u32x4*)dst, (const u32x4*)src, words,
                       (uint8_t*)dst + words * 16, (const uint8_t*)src + words * 16, tail);
    RS_HIP(hipGetLastError());
    return RADSORT_OK;
}

const char* radsort_strerror(int code)
{
    switch (code) {
    case RADSORT_OK: return "ok";
    case RADSORT_E_INVALID: return "invalid argument";
    case RADSORT_E_NOMEM: return "out of memory or workspace too small";
    case RADSORT_E_DEVICE: return hipGetErrorString(g_last_hip);
    case RADSORT_E_UNSUPPORTED: return "unsupported size or digit width";
    case RADSORT_E_TIMEOUT: return "a device-side check failed (a bounded wait gave up or an index left its range)";
    case RADSORT_E_ORDER: return "ordering check: a block was drawn before its loads were marked";
    default: return "unknown error";
    }
}

uint64_t radsort_segments_workspace_bytes(const uint64_t* offsets, uint32_t nseg, int key_bytes,
                                          int payload_bytes, const radsort_seg_tuning* tuning,
                                          const radsort_opts* opts)
{
    if (!offsets || (key_bytes != 4 && key_bytes != 8)) return 0;
    SegPlan P;
    if (make_seg_plan(P, offsets, nseg, key_bytes, payload_bytes, tuning, opts)) return 0;
    return P.total;
}

int radsort_sort_segments(void* keys, void* payload, const uint64_t* offsets,
                          const uint64_t* offsets_dev, uint32_t nseg, int key_bytes,
                          int payload_bytes, const radsort_seg_tuning* tuning,
                          const radsort_opts* opts, void* stream)
{
    if (!offsets || (nseg && !offsets_dev)) return RADSORT_E_INVALID;
    if (key_bytes != 4 && key_bytes != 8) return RADSORT_E_INVALID;
    if (payload_bytes != 0 && payload_bytes != 4 && payload_bytes != 8) return RADSORT_E_INVALID;
    if (nseg == 0 || offsets[nseg] == offsets[0]) return RADSORT_OK;
    int rc = check_args(keys, payload, offsets[nseg], payload_bytes);
    if (rc) return rc;
    SegPlan P;
    rc = make_seg_plan(P, offsets, nseg, key_bytes, payload_bytes, tuning, opts);
    if (rc) return rc;
    hipStream_t s = (hipStream_t)stream;
    uint8_t* ws = opts ? (uint8_t*)opts->workspace : nullptr;
    bool own = false;
    if (ws) {
        if (opts->workspace_bytes < P.total) return RADSORT_E_NOMEM;
    } else {
        hipError_t e = hipMalloc((void**)&ws, P.total);
        if (e != hipSuccess) {
            g_last_hip = e;
            return RADSORT_E_NOMEM;
        }
        own = true;
    }
    // [0]: small arrays, [1 + l]: lane l, [1 + kSegLanes]: the one-workgroup path,
    // [2 + kSegLanes]: its claim counter, [3 + kSegLanes]: the small arrays' claim counter
    uint32_t* err_small = (uint32_t*)ws;
    launch_fill(err_small, 4 + kSegLanes, 0, s);
    // the lanes fork first, so that their sorts run beside the batched kernels on the
    // caller's stream; they join back at the end
    LaneStreams* L = nullptr;
    if (!P.large.empty()) {
        rc = lane_streams(&L);
        if (!rc && hipEventRecord(L->fork, s) != hipSuccess) rc = RADSORT_E_DEVICE;
        for (uint32_t l = 0; !rc && l < kSegLanes; l++)
            if (hipStreamWaitEvent(L->s[l], L->fork, 0) != hipSuccess) rc = RADSORT_E_DEVICE;
        const uint64_t kb = key_bytes, vb = payload_bytes;
        for (size_t k = 0; !rc && k < P.large.size(); k++) {
            const uint32_t i = P.large[k], l = P.lane[k];
            void* kp = (uint8_t*)keys + offsets[i] * kb;
            void* vp = payload ? (uint8_t*)payload + offsets[i] * vb : nullptr;
            rc = run_one(kp, vp, offsets[i + 1] - offsets[i], key_bytes, payload_bytes,
                         P.choice[k], ws + P.lane_off[l], P.lane_bytes[l], err_small + 1 + l,
                         L->s[l]);
        }
    }
    if (!rc && (P.small_short || P.small_long)) {
        rc = dispatch<DoSmall>(key_bytes, payload_bytes, keys, payload, offsets_dev, nseg,
                               (uint64_t)0, P.small_short, P.small_long, err_small, err_small + 3 + kSegLanes, s);
    }
    if (!rc && P.wg_count) {
        rc = dispatch<DoWg>(key_bytes, payload_bytes, keys, payload, offsets_dev, nseg, P, ws,
                            err_small + 2 + kSegLanes, err_small + 1 + kSegLanes, s);
    }
    if (L) {
        for (uint32_t l = 0; l < kSegLanes; l++) {
            if (hipEventRecord(L->join[l], L->s[l]) != hipSuccess && !rc) rc = RADSORT_E_DEVICE;
            if (hipStreamWaitEvent(s, L->join[l], 0) != hipSuccess && !rc) rc = RADSORT_E_DEVICE;
        }
    }
    g_stats.timed = 0;
    g_stats.workspace_bytes = P.total;
    g_stats.input_bytes = (offsets[nseg] - offsets[0]) * (uint64_t)(key_bytes + payload_bytes);
    const bool check = opts && (opts->flags & RADSORT_F_CHECK);
    if (!rc && (check || own)) {
        // every lane's error word and the small kernel's
        uint32_t e = 0;
        std::vector<uint32_t> words(2 + kSegLanes, 0);
        RS_HIP(hipStreamSynchronize(s));
        RS_HIP(hipMemcpy(words.data(), err_small, 4 * words.size(), hipMemcpyDeviceToHost));
        for (uint32_t w : words) e |= w;
        g_stats.error_bits = e;
        if (e) rc = RADSORT_E_TIMEOUT;
    }
    if (own) {
        (void)hipStreamSynchronize(s);
        (void)hipFree(ws);
    }
    return rc;
}

}  // extern "C"

// ---- MSD-first split (Sec. 4.3, last paragraph) ------------------------------------
//
// One Radsort round on the most significant digit, finalized, leaves the array
// grouped by that digit (stably); each group is then an independent sort over the
// remaining digits, run as one batch of arrays by radsort_sort_segments (the
// digit that is now constant in every group costs no round there).  The group
// boundaries come from the digit totals that the round's counting pass leaves in
// the last row of the super-tile table, read back to the host before finalize
// reuses that memory.
int radsort_msd_sort_pairs(void* keys, void* payload, uint64_t n, int key_bytes,
                           int payload_bytes, int digit_bits, const radsort_opts* opts,
                           void* stream)
{
    int rc = check_args(keys, payload, n, payload_bytes);
    if (rc) return rc;
    if (opts && opts->workspace) return RADSORT_E_INVALID;  // the library sizes each phase
    Geo g;
    rc = make_geo(g, n, key_bytes, payload_bytes, digit_bits, opts);
    if (rc) return rc;
    if (n <= 1) return RADSORT_OK;
    radsort_opts o = opts ? *opts : radsort_opts{};
    o.flags &= ~(uint32_t)RADSORT_F_TIMING;
    radsort_state* st = nullptr;
    rc = radsort_state_create(&st, keys, payload, n, key_bytes, payload_bytes, digit_bits, &o);
    if (rc) return rc;
    st->dynamic = (o.flags & RADSORT_F_SHARED) || g.b <= 1024;
    st->shared = o.flags & RADSORT_F_SHARED;
    st->msd_shift = (int)(g.bits * (g.nt - 1));
    hipStream_t s = (hipStream_t)stream;
    std::vector<uint32_t> tot(g.sigma, 0);
    rc = radsort_state_setup(st, s);
    if (!rc) rc = radsort_state_round(st, s);
    if (!rc && hipMemcpyAsync(tot.data(), st->u32(st->L.stcnt) + (uint64_t)g.supers * g.sigma,
                              4ull * g.sigma, hipMemcpyDeviceToHost, s) != hipSuccess)
        rc = RADSORT_E_DEVICE;
    if (!rc) rc = radsort_state_finalize(st, s);
    if (!rc) rc = read_err(st, s, nullptr);  // waits: the totals are on the host
    const uint64_t radsort_ws = st->L.total;
    radsort_state_destroy(st);
    if (rc) return rc;
    std::vector<uint64_t> off(g.sigma + 1, 0);
    for (uint32_t d = 0; d < g.sigma; d++) off[d + 1] = off[d] + tot[d];
    if (off[g.sigma] != n) return RADSORT_E_DEVICE;  // never for a consistent round
    uint64_t* off_dev = nullptr;
    hipError_t e = hipMalloc((void**)&off_dev, 8ull * (g.sigma + 1));
    if (e != hipSuccess) {
        g_last_hip = e;
        return RADSORT_E_NOMEM;
    }
    rc = RADSORT_OK;
    if (hipMemcpyAsync(off_dev, off.data(), 8ull * (g.sigma + 1), hipMemcpyHostToDevice, s) !=
        hipSuccess)
        rc = RADSORT_E_DEVICE;
    radsort_opts so{};
    so.flags = o.flags & RADSORT_F_CHECK;
    if (!rc)
        rc = radsort_sort_segments(keys, payload, off.data(), off_dev, g.sigma, key_bytes,
                                   payload_bytes, nullptr, &so, stream);
    const uint64_t seg_ws = g_stats.workspace_bytes;
    (void)hipStreamSynchronize(s);  // off_dev is read by the segment kernels
    (void)hipFree(off_dev);
    g_stats.timed = 0;
    g_stats.workspace_bytes = std::max<uint64_t>(radsort_ws, seg_ws + 8ull * (g.sigma + 1));
    g_stats.input_bytes = n * (uint64_t)(key_bytes + payload_bytes);
    g_stats.rounds = g.nt;
    return rc;
}

// ---- the allocation-free entry point ----------------------------------------------
//
// radsort_sort_pairs_noalloc sorts with a workspace that is a file-scope device
// array, `scratch`, instead of a caller buffer or an allocation: each GPU the
// library runs on holds RADSORT_NOALLOC_SCRATCH_BYTES of it from the time the code
// object is loaded until the process ends.  In host code `scratch` names a host
// stand-in, never the device memory: its device address is looked up once per
// device (hipGetSymbolAddress, with that device current) and only that address is
// passed to kernels.  Every call on one GPU shares the array; the kernels clear
// what must start at zero (setup's fills), and calls that overlap on one GPU race.

static __device__ __align__(256) uint8_t scratch[RADSORT_NOALLOC_SCRATCH_BYTES];

namespace {

constexpr int kMaxScratchDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_dev[kMaxScratchDevices];  // device address of `scratch`, per device

// Device address of `scratch` on the current device (looked up on first use).
int scratch_address(void** out)
{
    int dev = 0;
    RS_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxScratchDevices) return RADSORT_E_UNSUPPORTED;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_dev[dev]) {
        void* p = nullptr;
        RS_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) return RADSORT_E_DEVICE;
        g_scratch_dev[dev] = p;
    }
    *out = g_scratch_dev[dev];
    return RADSORT_OK;
}

}  // namespace

int radsort_sort_pairs_noalloc(void* keys, void* payload, uint64_t n, int key_bytes,
                               int payload_bytes, int digit_bits, uint32_t block_elems,
                               uint32_t flags, void* stream)
{
    // timing records HIP events, which the library creates (allocates) on first use
    if (flags & RADSORT_F_TIMING) return RADSORT_E_INVALID;
    int rc = check_args(keys, payload, n, payload_bytes);
    if (rc) return rc;
    radsort_opts o{};
    o.block_elems = block_elems;
    o.flags = flags | RADSORT_F_SHARED;  // the launch forms below
    Geo g;
    rc = make_geo(g, n, key_bytes, payload_bytes, digit_bits, &o);
    if (rc) return rc;
    if (n <= 1) return RADSORT_OK;
    const Layout L = make_layout(g, false, true);
    if (L.total > (uint64_t)RADSORT_NOALLOC_SCRATCH_BYTES) return RADSORT_E_NOMEM;
    void* ws = nullptr;
    rc = scratch_address(&ws);
    if (rc) return rc;
    if (sort_is_small(g, &o)) {
        o.workspace = ws;
        o.workspace_bytes = RADSORT_NOALLOC_SCRATCH_BYTES;
        return sort_small(keys, payload, g, L, &o, (hipStream_t)stream);
    }
    radsort_state st;  // on the stack: nothing is allocated, on the host either
    st.g = g;
    st.L = L;
    st.ws = (uint8_t*)ws;
    st.own_ws = false;
    st.keys = keys;
    st.vals = payload;
    st.count = n;
    st.seq_draws = flags & RADSORT_F_SEQ_DRAWS;
    st.pack = true;
    // the launch forms that query no occupancy (the query's cache allocates)
    st.dynamic = true;
    st.shared = true;
    hipStream_t s = (hipStream_t)stream;
    const SegOne one = sort_in_workspace_plan(&st);
    if (one.shape >= 0) {
        rc = sort_in_workspace(&st, one, s);
    } else {
        rc = radsort_state_setup(&st, s);
        for (uint32_t r = 0; !rc && r < st.g.nt; r++) rc = radsort_state_round(&st, s);
        if (!rc) rc = radsort_state_finalize(&st, s);
    }
    g_stats.timed = 0;
    g_stats.workspace_bytes = L.total;
    g_stats.input_bytes = n * (uint64_t)(key_bytes + payload_bytes);
    g_stats.rounds = st.g.nt;
    if (!rc && (flags & RADSORT_F_CHECK)) rc = read_err(&st, s, nullptr);
    return rc;
}

#ifdef RS_TIMELINE
// Timeline builds only (not part of include/radsort.h): later Radsort rounds write
// kTlStamps real-time stamps per tile into buf (device memory of tiles * kTlStamps
// words), each round over the previous one.
extern "C" int radsort_timeline_buffer(void* buf, uint64_t tiles)
{
    g_tl = (uint64_t*)buf;
    g_tl_tiles = buf ? tiles : 0;
    return RADSORT_OK;
}
#endif
