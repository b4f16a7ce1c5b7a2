// All rounds of (update, associate) of one frame in one launch, for frames
// whose tiles are resident on the chip together.
//
// What bounds it: a round of a 640 x 480 frame is 2.3 us of distances in a
// launch of 7.5 us; the rest is the launch itself, fetching arguments and
// code anew, the pixels' loads, and global atomics that drain at its end.
// Here each workgroup keeps its tile's pixels in registers for all rounds and
// waits only for the tiles whose pixels can lie in its window's cells.
// With a launch per round and with this one, in us: 640 x 480 with 10 rounds
// 114 and 85, 1920 x 1080 280 and 226, 933 x 800 148 and 132, 320 x 240 with 5
// rounds 38 and 27, 1024 x 1024 with the convergence stop 122 and 94.
//
// Sums between rounds: every tile stores, for each cell of its window, the
// sums of its own pixels, and each tile adds up the few tiles that a cell's
// pixels can lie in.  No atomics and no clearing; integer sums, so the result
// is that of the launches one by one, bit for bit.  Two buffers, used in turn.
//
// Waiting.  Every stored word carries the round's number, and the reader
// loads a cell's words until all carry it: one trip through memory per round
// where a counter per tile (stores, wait for them, counter, wait for it,
// loads) took three, 1.4 to 1.9 us more per round.  The words are written and
// read as agent-scope relaxed atomics, which the XCDs' caches keep coherent.  A
// tile overwrites in round t what others read in round t - 1; it has then seen
// words of round t - 1 from each of them, which they store after they have
// read (who reads whom is symmetric: own cells at most two apart).
//
// Convergence stop: each tile also stores the shift of the centres it owns, as
// it stages them, in a word that carries the round; before the next round
// every workgroup adds up all tiles' words (stored half a round before) and
// takes the same decision.  Centres that come from the image move by less than
// 3 S <= 255 pixels or 256 units of colour, so the shifts of a window's at most
// 64 cells stay below 64 x 5 x 2^26 < 2^35.  A given centre may lie anywhere: a
// shift from 2^39 on goes whole into a second word, stored before the first,
// which then says so; the sums are those of 64-bit words in any case.
//
// Why every wait ends.  The launch does not assume that all its workgroups
// run at once.  Each workgroup registers (a bit in a census word) before its
// first store.  After its first tile it looks until every workgroup has
// registered or 20 us have passed; then it freezes the words that are not
// full, with the bits registered by then, in one atomic operation per word.
// So all workgroups agree on who was there in time.  If all were, each keeps
// its tile.  Else those in the census have done the first round of their own
// tiles, and every workgroup, also one that starts later, takes the other
// (round, tile) pairs from a common counter, the lower rounds first.  The lowest
// pair not yet done is then always a running workgroup's, and waits only for
// words of a round before, all done.  (With the convergence stop, a workgroup
// ends at the first pair it takes beyond the last round; a round has as many
// pairs as there are workgroups, so none takes one of the round after.)
// A frame alone on the chip never comes to that.  On a chip that several
// streams share the pairs cost as much as the kept tiles (1920 x 1080 14 us a
// round either way, 640 x 480 7.2 for 4.7), but a launch that fills the chip
// lets no other kernel in: us per frame on one, two and four streams, with a
// launch per round and with this one, 640 x 480 115, 66, 49 and 86, 50, 42;
// 1024 x 1024 156, 90, 71 and 133, 89, 90; 1920 x 1080 272, 194, 179 and 222,
// 228, 190.  (When late workgroups left, the few that were in time did the
// whole frame: 1920 x 1080 1,270 us on two streams.)
// All that supposes that nobody else writes the words.  Two calls in one
// workspace at once may clear them under a running launch; their results are
// then wrong, but no thread polls more than kPolls times.
#include "assign_tile.h"

#include <algorithm>

#pragma clang fp contract(off)

namespace slic {
namespace {

constexpr int kCensusBits = 31;    // workgroups per census word
constexpr int kCensusStride = 16;  // words (128 bytes) between census words
constexpr int kTicket = 8;         // word of the ticket counter, between two of them
constexpr int kMaxTiles = 1024;
constexpr int kMaxWords = (kMaxTiles + kCensusBits - 1) / kCensusBits;
constexpr long long kCensusTicks = 2000;  // of the 100 MHz clock: 20 us
constexpr unsigned long long kFrozen = 1ull << 63;
constexpr int kPolls = 1 << 23;  // of a thread in one launch: seconds
constexpr int kMaxCells = 64;                     // per window
// Tiles that a cell's sums are read from: a step of up to about half of the
// tile's height needs at most six.  The kernels for sixteen hold some forty
// registers more and read ten words more per round: with them alone a
// 1920 x 1080 frame takes 250 us for 226, 640 x 480 89.7 for 85.1 (320 x 240,
// whose cells have twelve, 26.9).
constexpr int kFewSources = 6, kMaxSources = 16;
constexpr int kCopies = 4;  // of the bins
// A stored word: the round (from 1) in its top 14 bits; below them a colour
// sum plus 2^40 (a tile's sums are below 2^37), or the position sums x, y (19
// bits each: at most 2048 pixels, offsets below 3 S <= 255) and the count.
constexpr int kTagShift = 18;  // in the high half
constexpr int kMaxRounds = (1 << 14) - 1;
constexpr int kPosBits = 19;
constexpr unsigned kPosMask = (1u << kPosBits) - 1;
constexpr long long kBias = 1ll << 40;
// A shift word: the round as above; below it a shift under kWideShift, or
// kWideMark: the shift is the tile's word in `wide`.  The narrow shifts of all
// tiles add up to less than kWideMark.
constexpr unsigned long long kPayload = (1ull << (32 + kTagShift)) - 1;
constexpr unsigned long long kWideShift = 1ull << 39, kWideMark = 1ull << 49;
static_assert(kMaxTiles * kWideShift <= kWideMark && kMaxTiles * kWideMark > kWideMark &&
                  kWideMark <= kPayload && 64ull * 5 * (1ull << 26) < kWideShift,
              "no sum of shifts reaches the round or the mark");

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

struct RoundsArgs {
    AssignImage g;
    unsigned long long* part;  // two buffers of part_words
    size_t part_words;
    int cw, cells;  // cells per row and per tile of the partial sums
    int nx;         // most tiles that a cell's neighbourhood meets in a row
    unsigned long long* census;  // zero before the launch, as are the partial sums
    int tiles_x, n_tiles;
    long long t0;     // first association of the launch
    int n;            // rounds, >= 2
    int store_last;   // the last round stores the labels
    int sums_last;    // the last round adds its sums to the ring
    long long limit;     // convergence stop: after a round whose shift is below it
    unsigned long long* shift;  // two buffers of n_tiles words, zero before the launch
    unsigned long long* wide;   // the same, not cleared: read only where a shift word says so
    int32_t* rounds_run;        // with converge (may be null)
    int polls;                  // after so many a thread waits no longer
};

template <class T>
__device__ __forceinline__ T agent_load(gmem<const T>* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <class T>
__device__ __forceinline__ void agent_store(gmem<T>* p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// n adjacent 32-bit words at p + i, of an array of `size`, in one store that the
// XCDs' caches keep coherent (word by word, the labels of one round of a
// 1024 x 1024 frame took 2 us more).
template <int n, class F>
__device__ __forceinline__ void store_through(int32_t* p, size_t size, size_t i, F word) {
    constexpr int kRaw = 0x27000, kAgent = 16;  // 32-bit elements; the sc1 bit
    const auto to = __builtin_amdgcn_make_buffer_rsrc(p, 0, static_cast<int>(size * 4), kRaw);
    const int at = static_cast<int>(i * 4);
    if constexpr (n == 4) {
        __builtin_amdgcn_raw_buffer_store_b128(u32x4{word(0), word(1), word(2), word(3)}, to, at, 0, kAgent);
    } else if constexpr (n == 2) {
        __builtin_amdgcn_raw_buffer_store_b64(u32x2{word(0), word(1)}, to, at, 0, kAgent);
    } else {
        __builtin_amdgcn_raw_buffer_store_b32(word(0), to, at, 0, kAgent);
    }
}

// Who takes part: waits for every workgroup to register, or freezes the
// census.  Leaves the participants' bits in `words` (all of them to see after
// the caller's barrier).
__device__ __forceinline__ void take_census(const RoundsArgs& a, long long ticks, unsigned* words) {
    const int lane = threadIdx.x;  // wave 0
    const int nwords = (a.n_tiles + kCensusBits - 1) / kCensusBits;
    gmem<unsigned long long>* const w = as_global(a.census) + lane * kCensusStride;
    const int in_word = min(a.n_tiles - lane * kCensusBits, kCensusBits);
    const unsigned full = in_word > 0 ? (1u << in_word) - 1u : 0u;
    const long long began = wall_clock64();
    unsigned bits = 0;
    for (;;) {
        bool ready = true;
        unsigned long long v = 0;
        if (lane < nwords) {
            v = agent_load<unsigned long long>(w);
            ready = (v & kFrozen) || static_cast<unsigned>(v) == full;
            bits = v & kFrozen ? static_cast<unsigned>(v >> 32) & 0x7FFFFFFFu
                               : static_cast<unsigned>(v);
        }
        if (__all(ready)) break;
        if (wall_clock64() - began < ticks) {
            __builtin_amdgcn_s_sleep(2);
            continue;
        }
        // each failed exchange means that a workgroup registered (at most 31
        // per word) or that the word is frozen
        while (!ready) {
            const unsigned long long frozen = v | kFrozen | ((v & 0x7FFFFFFFull) << 32);
            ready = __hip_atomic_compare_exchange_strong(w, &v, frozen, __ATOMIC_RELAXED,
                                                         __ATOMIC_RELAXED,
                                                         __HIP_MEMORY_SCOPE_AGENT) ||
                    (v & kFrozen) || static_cast<unsigned>(v) == full;
        }
    }
    if (lane < nwords) words[lane] = bits;
}

// SRC: most tiles that a cell's sums are read from.
template <int VEC, int ROWS, int DIST, int SRC, bool kConv>
__global__ __launch_bounds__(kThreads, 4) void rounds_kernel(RoundsArgs a) {
    using Sh = Shape<VEC, ROWS>;
    constexpr int kLogW = __builtin_ctz(Sh::kTileW), kLogH = __builtin_ctz(Sh::kTileH);
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ unsigned s_words[64];
    __shared__ int s_late, s_ticket;
    __shared__ unsigned long long s_shift, s_total[kThreads / 64];
    const AssignImage& g = a.g;
    const int S = g.S;
    const int me = blockIdx.x;
    const int tx = threadIdx.x % Sh::kTX, ty = threadIdx.x / Sh::kTX;
    const int comp = threadIdx.x & 3;
    gmem<long long>* const sums = as_global(g.sums);
    const size_t ring = static_cast<size_t>(g.K) * kSumStride;

    // ---- the tile at hand: its pixels and all that does not change from
    // round to round.  Four threads stage a window cell, one for each of
    // L, a, b and one for x, y and the count (the launch has at most 64 cells
    // per window, so one pass stages them all).
    float pl[ROWS][VEC], pa[ROWS][VEC], pb[ROWS][VEC];
    int x0, y0, gx_lo, gy_lo, ncx, ncells;
    int cx, cy, k;             // this thread's cell and its cluster (-1: none)
    bool owner;                // the cell's first pixel lies in the tile
    unsigned src[SRC];         // bytes from a buffer's start to the cell's sums, per tile
    unsigned valid;            // which of them are distinct tiles
    unsigned own_out;          // the same, to this tile's entry
    float v0, v1;              // the centre: this component; y
    auto enter = [&](int T) {
        const int by = T / a.tiles_x, bx = T - by * a.tiles_x;
        x0 = bx * Sh::kTileW;
        y0 = by * Sh::kTileH;
        {
            gmem<const float>* const Lg = as_global(g.L);
            gmem<const float>* const Ag = as_global(g.A);
            gmem<const float>* const Bg = as_global(g.B);
            const int xc = min(x0 + tx * VEC, g.w - VEC);  // outside: a clamped position
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
                const int y = min(y0 + ty * ROWS + r, g.h - 1);
                const size_t pi = static_cast<size_t>(y) * g.w + xc;
                if constexpr (VEC == 4) {
                    const float4 l4 = load_f4(Lg + pi), a4 = load_f4(Ag + pi), b4 = load_f4(Bg + pi);
                    pl[r][0] = l4.x; pl[r][1] = l4.y; pl[r][2] = l4.z; pl[r][3] = l4.w;
                    pa[r][0] = a4.x; pa[r][1] = a4.y; pa[r][2] = a4.z; pa[r][3] = a4.w;
                    pb[r][0] = b4.x; pb[r][1] = b4.y; pb[r][2] = b4.z; pb[r][3] = b4.w;
                } else if constexpr (VEC == 2) {
                    const vf2 l2 = load_f2(Lg + pi), a2 = load_f2(Ag + pi), b2 = load_f2(Bg + pi);
                    pl[r][0] = l2.x; pl[r][1] = l2.y;
                    pa[r][0] = a2.x; pa[r][1] = a2.y;
                    pb[r][0] = b2.x; pb[r][1] = b2.y;
                } else {
                    pl[r][0] = Lg[pi];
                    pa[r][0] = Ag[pi];
                    pb[r][0] = Bg[pi];
                }
            }
        }
        gx_lo = g.by_S.quotient(x0) - 1;
        gy_lo = g.by_S.quotient(y0) - 1;
        const int gx_hi = g.by_S.quotient(min(x0 + Sh::kTileW, g.w) - 1) + 1;
        const int gy_hi = g.by_S.quotient(min(y0 + Sh::kTileH, g.h) - 1) + 1;
        ncx = gx_hi - gx_lo + 1;
        ncells = ncx * (gy_hi - gy_lo + 1);
        // row of cell i: floor((i + 1/2) / ncx) through the hardware
        // reciprocal; for i < 64 the product is within 2^-15 of the quotient,
        // which lies at least 1/128 from an integer
        const int i = threadIdx.x >> 2;
        const int row = static_cast<int>((static_cast<float>(i) + 0.5f) *
                                         __builtin_amdgcn_rcpf(static_cast<float>(ncx)));
        cx = gx_lo + (i - row * ncx);
        cy = gy_lo + row;
        const bool live = i < ncells && cx >= 0 && cy >= 0 && cx < g.ns_c && cy < g.ns_r;
        k = live ? cy * g.ns_c + cx : -1;
        owner = live && cx * S >> kLogW == bx && cy * S >> kLogH == by;
        own_out = (static_cast<unsigned>(T * a.cells + row * a.cw + (i - row * ncx)) * 4 + comp) * 8;
        const int ccx = live ? cx : 0, ccy = live ? cy : 0;
        const int px0 = max((ccx - 1) * S, 0) >> kLogW, px1 = (min((ccx + 2) * S, g.w) - 1) >> kLogW;
        const int py0 = max((ccy - 1) * S, 0) >> kLogH, py1 = (min((ccy + 2) * S, g.h) - 1) >> kLogH;
        valid = 0;
        int b = 0, r = 0;  // source m is tile (px0 + b, py0 + r)
#pragma unroll
        for (int m = 0; m < SRC; ++m) {
            const bool ok = px0 + b <= px1 && py0 + r <= py1;
            const int ptx = ok ? px0 + b : px0, pty = ok ? py0 + r : py0;
            const int cell = (ccy + 1 - g.by_S.quotient(pty << kLogH)) * a.cw + ccx + 1 -
                             g.by_S.quotient(ptx << kLogW);
            src[m] = (static_cast<unsigned>((pty * a.tiles_x + ptx) * a.cells + cell) * 4 + comp) * 8;
            valid |= ok ? 1u << m : 0u;
            if (++b == a.nx) {
                b = 0;
                ++r;
            }
        }
    };
    auto load_centre = [&]() {
        gmem<float>* const c = as_global(g.cen) + static_cast<size_t>(max(k, 0)) * kCenStride;
        v0 = agent_load<float>(c + comp);
        v1 = agent_load<float>(c + 4);
    };
    enter(me);

    // ---- register
    if (threadIdx.x == 0) {
        const unsigned long long v = __hip_atomic_fetch_or(
            as_global(a.census) + (me / kCensusBits) * kCensusStride, 1ull << (me % kCensusBits),
            __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        s_late = (v & kFrozen) && !((v >> (32 + me % kCensusBits)) & 1ull);
        s_shift = 0;
    }
    load_centre();
    __syncthreads();
    const bool late = __builtin_amdgcn_readfirstlane(s_late) != 0;
    const unsigned long long mask =  // the summed fields of this thread's words
        comp < 3 ? (1ull << (32 + kTagShift)) - 1
                 : (1ull << (32 + kTagShift)) - 1 - (static_cast<unsigned long long>(kPosMask) << kPosBits);

    bool all_here = true;  // false: the census was frozen
    int absent = 0;        // workgroups not in it
    int taken = 0;         // pairs from the counter
    int polls = a.polls;   // left to this thread
    int T = me;
    int round = 0;  // association a.t0 + round
    int checked = 0;  // rounds whose shift has been looked at
    // One round of the tile at hand; false: the rounds before were the last.
    auto pass = [&]() {
        if constexpr (kConv) {
            if (round > checked) {
                // the shift of the round before, from all tiles
                const size_t buffer = (round & 1) ? 0 : a.n_tiles;
                gmem<const unsigned long long>* const in =
                    as_global(static_cast<const unsigned long long*>(a.shift)) + buffer;
                gmem<const unsigned long long>* const wide =
                    as_global(static_cast<const unsigned long long*>(a.wide)) + buffer;
                auto sum_of_tiles = [&](auto shift_of) {
                    unsigned long long mine = 0;
                    for (int j = threadIdx.x; j < a.n_tiles; j += kThreads) mine += shift_of(j);
                    for (int d = 32; d > 0; d >>= 1) mine += __shfl_xor(mine, d);
                    if ((threadIdx.x & 63) == 0) s_total[threadIdx.x >> 6] = mine;
                    __syncthreads();
                    unsigned long long total = 0;
#pragma unroll
                    for (int q = 0; q < kThreads / 64; ++q) total += s_total[q];
                    return total;
                };
                unsigned long long total = sum_of_tiles([&](int j) {
                    unsigned long long v;
                    while ((v = agent_load<unsigned long long>(in + j)) >> (32 + kTagShift) !=
                               static_cast<unsigned>(round) &&
                           --polls > 0) {
                    }
                    return v & kPayload;
                });
                if (total >= kWideMark) {  // again, with the marked tiles' own words
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
                    __syncthreads();  // s_total is read
                    total = sum_of_tiles([&](int j) {
                        const unsigned long long v = agent_load<unsigned long long>(in + j) & kPayload;
                        return v == kWideMark ? agent_load<unsigned long long>(wide + j) : v;
                    });
                }
                if (static_cast<long long>(total) < a.limit) {
                    if (T == 0 && threadIdx.x == 0 && a.rounds_run) *a.rounds_run = round;
                    return false;
                }
                checked = round;
            }
        }
        const long long t = a.t0 + round;
        float4* const cen4 = reinterpret_cast<float4*>(smem);
        float* const cenf = reinterpret_cast<float*>(smem);
        float* const ceny = reinterpret_cast<float*>(cen4 + ncells);
        int* const kidx = reinterpret_cast<int*>(ceny + ncells);
        unsigned long long* const bins =
            reinterpret_cast<unsigned long long*>(smem + static_cast<size_t>(ncells) * 24);
        const bool last = round == a.n - 1;
        const bool sums_out = !last || a.sums_last;
        const int i = threadIdx.x >> 2;

        // ---- the window's centres
        if (i < ncells) {
            long long s0 = 0, s1 = 0, n = 0;
            if (round > 0 && k >= 0) {  // (no words to wait for where there is no centre)
                gmem<const char>* const in = reinterpret_cast<gmem<const char>*>(
                    as_global(a.part) + ((round & 1) ? 0 : a.part_words));
                unsigned long long w[SRC];
                for (;;) {
#pragma unroll
                    for (int m = 0; m < SRC; ++m) {
                        // (opaque: the sums base + offset would be kept in
                        // two registers each through the loop)
                        unsigned place = src[m];
                        asm volatile("" : "+v"(place));
                        w[m] = agent_load<unsigned long long>(
                            reinterpret_cast<gmem<const unsigned long long>*>(in + place));
                    }
                    unsigned off = 0;  // any bit: a word of another round
#pragma unroll
                    for (int m = 0; m < SRC; ++m)
                        off |= static_cast<unsigned>(w[m] >> 32) ^ (static_cast<unsigned>(round) << kTagShift);
                    if ((off >> kTagShift) == 0 || --polls <= 0) break;
                }
                unsigned long long sum = 0;
                unsigned sum_y = 0;
#pragma unroll
                for (int m = 0; m < SRC; ++m) {
                    const unsigned long long u = (valid >> m) & 1u ? w[m] : 0ull;
                    sum += u & mask;
                    sum_y += static_cast<unsigned>(u >> kPosBits) & kPosMask;
                }
                // the count is in the fourth thread's sum (the four threads of
                // a cell are here together)
                n = __builtin_amdgcn_mov_dpp(static_cast<int>(sum >> (2 * kPosBits)), 0xFF, 0xF, 0xF,
                                             true);
                s0 = comp < 3 ? static_cast<long long>(sum) - __popc(valid) * kBias
                              : static_cast<long long>(sum & ((1ull << (2 * kPosBits)) - 1)) +
                                    n * ((cx - 1) * S);
                s1 = static_cast<long long>(sum_y) + n * ((cy - 1) * S);
            } else if (a.t0 > 0 && k >= 0) {
                gmem<const long long>* const sp = sums + ring * static_cast<size_t>((t + 2) % 3) +
                                                  static_cast<size_t>(k) * kSumStride;
                s0 = sp[comp];
                s1 = sp[4];
                n = sp[5];
            }
            // With a frozen census the centre of the round before may come from
            // another workgroup.  Its owner stored it before the word of that
            // round seen above, so only a load after the wait is sure to find
            // it.  (A centre stored in this round has pixels: v0, v1 are not
            // used then.)
            if (!all_here) {
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");  // (keeps the order)
                load_centre();
            }
            const double dn = static_cast<double>(n > 0 ? n : 1);
            const double inv = 1.0 / static_cast<double>(1 << kQShift);
            const double q0 = static_cast<double>(s0) / dn;
            const double q1 = static_cast<double>(s1) / dn;
            // a centre with no pixels keeps its value
            if constexpr (kConv) {  // L1 shift, each component rint(|d| 2^18)
                if (owner && n > 0) {
                    const double q = static_cast<double>(1 << kQShift);
                    const float m0 = static_cast<float>(comp < 3 ? q0 * inv : q0);
                    long long d = llrint(fabs(static_cast<double>(m0) - v0) * q);
                    if (comp == 3)
                        d += llrint(fabs(static_cast<double>(static_cast<float>(q1)) - v1) * q);
                    if (d) atomicAdd(&s_shift, static_cast<unsigned long long>(d));
                }
            }
            v0 = n > 0 ? static_cast<float>(comp < 3 ? q0 * inv : q0) : v0;
            v1 = n > 0 ? static_cast<float>(q1) : v1;
            // where there is no centre, an infinite colour distance never wins
            cenf[i * 4 + comp] = k >= 0 ? v0 : comp == 0 ? __builtin_huge_valf() : 0.0f;
            if (comp == 3) {
                ceny[i] = k >= 0 ? v1 : 0.0f;
                kidx[i] = k;
            }
            if (owner) {
                if (n > 0) {
                    gmem<float>* const c = as_global(g.cen) + static_cast<size_t>(k) * kCenStride;
                    agent_store<float>(c + comp, v0);
                    if (comp == 3) agent_store<float>(c + 4, v1);
                }
                if ((kConv || last) && t > 0 && comp == 3)
                    agent_store<int32_t>(as_global(g.counts) + k, static_cast<int32_t>(n));
                if (a.sums_last && round >= a.n - 2) {
                    // the ring's accumulators of the last round and of the
                    // launch after it
                    gmem<long long>* const z = sums + ring * static_cast<size_t>((t + 1) % 3) +
                                               static_cast<size_t>(k) * kSumStride;
                    agent_store<long long>(z + comp, 0);
                    if (comp < 2) agent_store<long long>(z + 4 + comp, 0);
                }
            }
        }
        if (sums_out)
            for (int j = threadIdx.x; j < kCopies * bin_stride(ncells); j += kThreads) bins[j] = 0ull;
        __syncthreads();
        if constexpr (kConv) {
            if (threadIdx.x == 0) {  // (the next additions are two barriers away)
                const size_t at = ((round & 1) ? a.n_tiles : 0) + T;
                unsigned long long v = s_shift;
                if (v >= kWideShift) {
                    agent_store<unsigned long long>(as_global(a.wide) + at, v);
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
                    v = kWideMark;
                }
                agent_store<unsigned long long>(
                    as_global(a.shift) + at,
                    v | (static_cast<unsigned long long>(round + 1) << (32 + kTagShift)));
                s_shift = 0;
            }
        }

        // ---- associate, labels, sums
        const int x = x0 + tx * VEC, yb = y0 + ty * ROWS;
        const bool col_ok = x < g.w;
        const int gx_rel = g.by_S.quotient(col_ok ? x : x0) - gx_lo - 1;
        int cellv[ROWS][VEC];
        find_cells<VEC, ROWS, DIST>(cen4, ceny, kidx, ncx, gx_rel, gy_lo, g, x, yb, pl, pa, pb, cellv);
        if ((kConv || last) && a.store_last) {  // any round may turn out the last
            gmem<int32_t>* const labels = as_global(g.labels);
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
                if (!col_ok || yb + r >= g.h) continue;
                const size_t pi = static_cast<size_t>(yb + r) * g.w + x;
                if (kConv && (round == 0 || !all_here)) {
                    // (the next round's may come from another workgroup: these
                    // are in memory before this round's words)
                    store_through<VEC>(g.labels, static_cast<size_t>(g.w) * g.h, pi, [&](int v) {
                        return static_cast<unsigned>(kidx[cellv[r][v]]);
                    });
                } else if constexpr (VEC == 4) {
                    store_i4(labels + pi, kidx[cellv[r][0]], kidx[cellv[r][1]], kidx[cellv[r][2]],
                             kidx[cellv[r][3]]);
                } else if constexpr (VEC == 2) {
                    store_i2(labels + pi, kidx[cellv[r][0]], kidx[cellv[r][1]]);
                } else {
                    labels[pi] = kidx[cellv[r][0]];
                }
            }
        }
        if (sums_out) {
            accumulate<VEC, ROWS>(bins + (threadIdx.x & (kCopies - 1)) * bin_stride(ncells), ncells,
                                  cellv, pl, pa, pb, tx * VEC, ty * ROWS, col_ok ? g.h - yb : 0);
            if (kConv && (round == 0 || !all_here)) __builtin_amdgcn_s_waitcnt(0);
            __syncthreads();
            if (i < ncells) {
                unsigned long long p = 0;
#pragma unroll
                for (int c = 0; c < kCopies; ++c)
                    p += bins[c * bin_stride(ncells) + comp * ncells + i];
                const long long n = static_cast<long long>(p >> 48);  // of the position word
                if (!last) {
                    if (comp < 3) {
                        p += kBias;
                    } else {
                        // positions from the corner of the cell's neighbourhood
                        const long long px = static_cast<long long>(p & 0xFFFFFFull) + n * (x0 - (cx - 1) * S);
                        const long long py =
                            static_cast<long long>((p >> 24) & 0xFFFFFFull) + n * (y0 - (cy - 1) * S);
                        p = static_cast<unsigned long long>(px) |
                            (static_cast<unsigned long long>(py) << kPosBits) |
                            (static_cast<unsigned long long>(n) << (2 * kPosBits));
                    }
                    p |= static_cast<unsigned long long>(round + 1) << (32 + kTagShift);
                    // before another tile sees this word: the ring's
                    // accumulators cleared here, to which it may add, and (with
                    // a frozen census) the centre stored here, which it may load
                    if (round == 0 || !all_here || (a.sums_last && round == a.n - 2))
                        __builtin_amdgcn_s_waitcnt(0);
                    gmem<char>* const out = reinterpret_cast<gmem<char>*>(
                        as_global(a.part) + ((round & 1) ? a.part_words : 0));
                    agent_store<unsigned long long>(
                        reinterpret_cast<gmem<unsigned long long>*>(out + own_out), p);
                } else if (p != 0) {
                    gmem<unsigned long long>* const z = reinterpret_cast<gmem<unsigned long long>*>(
                        sums + ring * static_cast<size_t>(t % 3) + static_cast<size_t>(k) * kSumStride);
                    auto add = [&](int j, unsigned long long v) {
                        __hip_atomic_fetch_add(z + j, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    };
                    if (comp < 3) {
                        add(comp, p);
                    } else {
                        add(3, static_cast<unsigned long long>(
                                   static_cast<long long>(p & 0xFFFFFFull) + n * x0));
                        add(4, static_cast<unsigned long long>(
                                   static_cast<long long>((p >> 24) & 0xFFFFFFull) + n * y0));
                        add(5, static_cast<unsigned long long>(n));
                    }
                }
            }
        }
        __syncthreads();  // the bins are read
        if constexpr (kConv) {
            if (last && T == 0 && threadIdx.x == 0 && a.rounds_run) *a.rounds_run = a.n;
        }
        return true;
    };
    for (bool first = true;; first = false) {
        if (!(first && late) && !pass()) break;
        if (first) {
            if (threadIdx.x < 64) take_census(a, late ? 0 : kCensusTicks, s_words);
            __syncthreads();
            absent = a.n_tiles;
            for (int j = 0; j * kCensusBits < a.n_tiles; ++j)
                absent -= __popc(__builtin_amdgcn_readfirstlane(s_words[j]));
            all_here = absent == 0;
        }
        if (all_here) {  // the same tile again
            if (++round == a.n) break;
            continue;
        }
        // the next pair that nobody has: the first round of the absent
        // workgroups' tiles, then round by round all tiles; a.n at most, a
        // workgroup's share, so that the chip's other users come in between
        if (taken++ == a.n) break;
        if (threadIdx.x == 0)
            s_ticket = static_cast<int>(__hip_atomic_fetch_add(as_global(a.census) + kTicket, 1ull,
                                                               __ATOMIC_RELAXED,
                                                               __HIP_MEMORY_SCOPE_AGENT));
        __syncthreads();
        // (unsigned: in range for any value of the counter)
        unsigned q = __builtin_amdgcn_readfirstlane(s_ticket);
        const unsigned tiles = a.n_tiles;
        if (absent <= 0 || q >= static_cast<unsigned>(absent)) {
            q -= absent;
            const unsigned r = q / tiles + 1u;
            if (r >= static_cast<unsigned>(a.n)) break;
            round = r;
            T = q % tiles;
        } else {
            round = 0;
            for (int j = 0;; ++j) {
                const int in_word = min(a.n_tiles - j * kCensusBits, kCensusBits);
                unsigned missing = ((1u << in_word) - 1u) &
                                   ~__builtin_amdgcn_readfirstlane(s_words[j]);
                const unsigned c = __popc(missing);
                if (q >= c) {
                    q -= c;
                    continue;
                }
                while (q--) missing &= missing - 1u;
                T = j * kCensusBits + __builtin_ctz(missing);
                break;
            }
        }
        enter(T);
    }
}

__global__ __launch_bounds__(256) void clear_words_kernel(uint4* p, size_t n) {
    const size_t i = static_cast<size_t>(blockIdx.x) * 256 + threadIdx.x;
    if (i < n) p[i] = make_uint4(0u, 0u, 0u, 0u);
}

// A census frozen from the start, without the workgroups that `absent` names.
__global__ __launch_bounds__(64) void freeze_census_kernel(unsigned long long* census, int n_tiles,
                                                           uint32_t absent) {
    const int in_word = min(n_tiles - static_cast<int>(threadIdx.x) * kCensusBits, kCensusBits);
    if (in_word <= 0) return;
    const unsigned here = ((1u << in_word) - 1u) & ~absent;
    census[threadIdx.x * kCensusStride] = kFrozen | (static_cast<unsigned long long>(here) << 32);
}

template <int VEC, int ROWS, int DIST, int SRC, bool kConv>
hipError_t launch_rounds_as(const RoundsArgs& a, hipStream_t s) {
    KernelTimer timer("assign_rounds", s);
    rounds_kernel<VEC, ROWS, DIST, SRC, kConv>
        <<<a.n_tiles, kThreads, assign_lds_bytes(kMaxCells, kCopies), s>>>(a);
    return hipGetLastError();
}

using RoundsFn = hipError_t (*)(const RoundsArgs&, hipStream_t);

// By distance, number of sources and the convergence stop.
template <int VEC, int ROWS>
RoundsFn shape_fn(int dist, int sources, bool conv) {
    constexpr int F = kFewSources, M = kMaxSources;
    static constexpr RoundsFn fn[2][2][2] = {
        {{launch_rounds_as<VEC, ROWS, 0, F, false>, launch_rounds_as<VEC, ROWS, 0, F, true>},
         {launch_rounds_as<VEC, ROWS, 0, M, false>, launch_rounds_as<VEC, ROWS, 0, M, true>}},
        {{launch_rounds_as<VEC, ROWS, 1, F, false>, launch_rounds_as<VEC, ROWS, 1, F, true>},
         {launch_rounds_as<VEC, ROWS, 1, M, false>, launch_rounds_as<VEC, ROWS, 1, M, true>}}};
    return fn[dist ? 1 : 0][sources > F ? 1 : 0][conv ? 1 : 0];
}

RoundsFn rounds_fn(int variant, int dist, int sources, bool conv) {
    switch (variant) {  // the association's variants, in their order
        case 1: return shape_fn<1, 1>(dist, sources, conv);
        case 2: return shape_fn<1, 2>(dist, sources, conv);
        case 3: return shape_fn<1, 4>(dist, sources, conv);
        case 4: return shape_fn<4, 1>(dist, sources, conv);
        case 5: return shape_fn<4, 2>(dist, sources, conv);
        case 6: return shape_fn<2, 1>(dist, sources, conv);
        case 7: return shape_fn<2, 2>(dist, sources, conv);
        default: return nullptr;
    }
}

size_t clear_words(const RoundsArgs& a) {
    // census, shifts (an even number of words), partial sums
    return (static_cast<size_t>(kMaxWords) * kCensusStride + 2 * static_cast<size_t>(a.n_tiles) +
            2 * a.part_words) * 2;
}

// The launch's arguments for a variant's tiles; false where the frame does
// not suit: more tiles than are resident at once (four workgroups per compute
// unit), a step whose cluster sums do not fit the packed word (S <= 85: 9 S^2
// pixels, offsets below 3 S), windows of more than 64 cells, cells that meet
// more than 16 tiles, or arrays larger than the connectivity buffers they are
// laid in.
bool rounds_args(const Workspace& ws, int32_t w, int32_t h, const Grid& g, int variant, int cus,
                 RoundsArgs* a, int* sources) {
    int tw = 0, th = 0;
    const int S = g.S;
    if (S > 85 || !assign_variant_supported(variant, w, h, S) ||
        !assign_variant_shape(variant, nullptr, nullptr, &tw, &th))
        return false;
    const int tiles_x = (w + tw - 1) / tw, tiles_y = (h + th - 1) / th;
    if (static_cast<long long>(tiles_x) * tiles_y > std::min(kMaxTiles, 4 * cus)) return false;
    a->tiles_x = tiles_x;
    a->n_tiles = tiles_x * tiles_y;
    auto gcd = [](int u, int v) {
        while (v) {
            const int r = u % v;
            u = v;
            v = r;
        }
        return u;
    };
    // most tiles met by n pixels that start at a multiple of `step`, and most
    // cells that a tile meets
    auto most = [&](int tile, int step, int n) { return (tile - gcd(tile, step) + n - 1) / tile + 1; };
    auto cells = [&](int tile) { return (S - gcd(tile, S) + tile - 1) / S + 1; };
    const int cw = cells(tw), ch = cells(th);
    a->nx = std::min(most(tw, S, 3 * S), tiles_x);
    const int ny = std::min(most(th, S, 3 * S), tiles_y);
    *sources = a->nx * ny;
    a->cw = cw + 2;  // the window has a ring of cells around the tile's own
    a->cells = a->cw * (ch + 2);
    if (*sources > kMaxSources || a->cells > kMaxCells) return false;
    a->part_words = static_cast<size_t>(a->n_tiles) * a->cells * 4;
    // the connectivity buffers are free until the clean-up: census and partial
    // sums lie in the ranks and local roots (adjacent arrays)
    // (and the shifts too wide for their words in the labels' parents)
    const size_t n = static_cast<size_t>(w) * h * sizeof(int32_t);
    a->wide = reinterpret_cast<unsigned long long*>(ws.ccl0);
    if (2 * static_cast<size_t>(a->n_tiles) * sizeof(unsigned long long) > n) return false;
    a->census = reinterpret_cast<unsigned long long*>(ws.ccl2);
    a->shift = a->census + kMaxWords * kCensusStride;
    a->part = a->shift + 2 * a->n_tiles;
    return clear_words(*a) * sizeof(uint32_t) <= 2 * n;
}

}  // namespace

// A variant that the caller chose keeps its tiles.  The built-in choice is one
// for launches of single rounds; here small tiles pay longer, as nothing is
// loaded or launched per round and a frame's slowest compute unit sets its
// pace.  Per round, in us: 320 x 240 3.06 with 32 x 8 tiles, 3.15 with 32 x 16,
// 3.93 with 64 x 16; 640 x 480 4.24 with 32 x 16, 5.05 with 64 x 16 (300 tiles
// on 256 units); 1024 x 1024 7.6 with 64 x 32, 8.9 with 64 x 16.
// More than 2.5 tiles per unit only where no larger tile of the table avoids
// it: up to there two frames on different streams run side by side, beyond
// it one waits for the other.  A frame of ten rounds with clean-up, in us, on
// one and on four streams: 720 x 576 97 and 85 with 32 x 16 tiles (828), 102
// and 40 with 32 x 32 (414); 1280 x 720 131 and 139 with 64 x 16 (900), 137 and
// 84 with 64 x 32 (460).
int rounds_variant(const Workspace& ws, int32_t w, int32_t h, const Grid& g, int variant, int n) {
    if (n < kMinRounds || n > kMaxRounds) return 0;
    RoundsArgs a;
    int sources = 0;
    const long long px = static_cast<long long>(w) * h;
    const int cus = compute_units();
    auto fits = [&](int v) { return rounds_args(ws, w, h, g, v, cus, &a, &sources); };
    if (variant != assign_default_variant(w, h, g.S)) return fits(variant) ? variant : 0;
    const int small[] = {1, 2, variant};  // by the frame's size
    const int first = px <= (1ll << 17) ? 0 : px <= (1ll << 19) ? 1 : 2;
    for (const int v : {small[first], std::max(small[first], 2), 3, 5})
        if (fits(v) && 2 * a.n_tiles <= 5 * cus) return v;
    for (int i = first; i < 3; ++i)
        if (fits(small[i])) return small[i];
    return 0;
}

uint32_t* rounds_clear(const Workspace& ws, int32_t w, int32_t h, const Grid& g, int variant,
                       size_t* words) {
    RoundsArgs a;
    int sources = 0;
    if (!rounds_args(ws, w, h, g, variant, compute_units(), &a, &sources)) return nullptr;
    *words = clear_words(a);
    return reinterpret_cast<uint32_t*>(a.census);
}

hipError_t launch_rounds(const Workspace& ws, int32_t w, int32_t h, const Grid& g, int64_t t0, int n,
                         int variant, bool store_last, bool sums_last, bool cleared, hipStream_t s,
                         const RoundsStop* stop, const RoundsTest* test) {
    RoundsArgs a;
    int sources = 0;
    const int cus = compute_units();
    if (n < 2 || n > kMaxRounds || !rounds_args(ws, w, h, g, variant, cus, &a, &sources))
        return hipErrorInvalidValue;
    // workgroups said to take part must be able to run together
    if (test && (a.n_tiles > 2 * cus ||
                 !(((1u << std::min(a.n_tiles, kCensusBits)) - 1u) & ~test->absent)))
        return hipErrorInvalidValue;
    a.g = assign_image(ws, w, h, g, variant);
    a.t0 = t0;
    a.n = n;
    a.store_last = store_last;
    a.sums_last = sums_last;
    if (!cleared) {
        const size_t words = clear_words(a);
        KernelTimer timer("assign_clear", s);
        clear_words_kernel<<<static_cast<unsigned>((words + 1023) / 1024), 256, 0, s>>>(
            reinterpret_cast<uint4*>(a.census), words / 4);
    }
    if (test) freeze_census_kernel<<<1, 64, 0, s>>>(a.census, a.n_tiles, test->absent);
    a.polls = test && test->polls > 0 ? test->polls : kPolls;
    a.limit = stop ? stop->limit : 0;
    a.rounds_run = stop ? stop->rounds_run : nullptr;
    return rounds_fn(variant, g.dist, sources, stop != nullptr)(a, s);
}

}  // namespace slic
