// GPU entropy decoding of many baseline scans.
//
// The host plans the work: it checks every job, builds its Huffman tables in
// the layouts that the kernels copy to LDS, lists the restart intervals
// (sorted by length within a job) and chooses which of them are split.  A
// launch then runs, on one stream:
//   entropy_destuff         the intervals' bytes without stuffed zeros, into
//                           the batch's own memory (entropy_destuff_count
//                           first, where an interval takes several waves);
//   entropy_guess, _follow, where intervals are split: the block boundaries,
//   _resolve                block counts and DC predictions at which their
//                           parts begin;
//   entropy_decode<true>    the parts of split intervals, a lane each;
//   entropy_decode<false>   the other intervals, a lane each (in passes, where
//                           their destuffed bytes exceed kPassBytes).
// Both decoding kernels write whole blocks in MCU order, the layout that
// mjd_decode reads.  Each interval's status goes to a device array.
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <new>
#include <string>
#include <vector>

#include "entropy_walk.h"
#include "host_jpeg.h"
#include "mjd_internal.h"

namespace mjd {
namespace gent {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
constexpr uint64_t kMaxStream = 0xFFFFFF00u;  // stream offsets are 32-bit
constexpr uint32_t kTile = 4096;              // raw bytes that one wave destuffs
constexpr uint32_t kLongSplit = 512;          // chunks above which a workgroup resolves an interval
constexpr uint32_t kTail = 8192;              // bytes past the chunks that a workgroup may copy
constexpr uint32_t kPad = 48;                 // bytes past an interval's raw length in its region
constexpr uint32_t kMended = 4, kCounters = 5;  // the counter of the breaks that a launch has mended; counters
constexpr uint32_t kStatusOk = 0xFFFFFFFFu;   // else (block in the interval) << 2 | kBadCode, kBadRun or kOverrun

struct GJob {
  const uint8_t* jpg;
  int16_t* coef;
  const FastTables* tables;
  const GCodes* codes;  // the same tables' canonical codes
  uint16_t* skip;      // kTableSlots skip tables, where the job has split intervals
  uint32_t bpm;        // blocks per MCU
  uint32_t comp_bits;  // component of block b of an MCU in bits 2b..2b+1
  uint32_t dc_slots;   // its DC and AC table slots, likewise
  uint32_t ac_slots;
};

// One restart interval: its entropy-coded bytes [start, end) of the stream
// (end: the marker that closes it), where its destuffed bytes go (16-byte
// units), and its blocks among the job's.
struct GInterval {
  uint32_t start, end;
  uint32_t dst;
  uint32_t block0, n_blocks;
  uint32_t job;
};

// A tile of an interval longer than kTile; first: the interval's first tile
// among the pass's.
struct GTile {
  uint32_t iv, index, first;
};

// An interval decoded by chunks of destuffed bytes.  Chunks are numbered over
// the batch, a job's one after the other, and lie in that order in memory.
// 128 bytes: a 12-image corpus of 4:2:0 files takes 322 us (330 with 64, 421
// with 256, 595 with 512), a 4000x3000 file with markers per row 162 (134, 263,
// 445).  Shorter ones leave more boundaries unguessed: a noisy 1024x768 file
// without markers has 12 broken chains at quality 95 (265 with 64, none with
// 256) and takes 0.59 ms (6.3, 0.31), and at 98 462 (1702, 33) and 18 ms (60, 2.1).
constexpr uint32_t kChunk = 128, kChunkWords = kChunk / 4;
struct GSplit {
  uint32_t iv, chunk0, n_chunks;
};
// A workgroup's share of the chunks, of one job.
struct GGroup {
  uint32_t job, first, count;
};

// The part of the decoding that begins in one half of a chunk.
constexpr uint32_t kParts = 2, kPart = kChunk / kParts;  // entropy_follow counts two
struct GTask {
  uint32_t iv;
  uint32_t word, bit_b;  // where it starts: word, bit | first block of the MCU << 8
  uint32_t block0, n_blocks;
  uint16_t dc[3];
  uint16_t pad[3];
};
static_assert(sizeof(GTask) == 32, "two 16-byte loads");

// What a lane found from the start of a part to the first block boundary in
// the next: blocks and DC differences, and that boundary.
struct GHop {
  uint16_t blocks;
  uint16_t dc[3];
  uint32_t state;
  uint32_t pad;
};
static_assert(sizeof(GHop) == 16, "one 16-byte store");

// Tasks, or intervals, of one job that a workgroup decodes.
struct GItem {
  uint32_t job, first, count;
  uint32_t bytes;  // of its longest lane
};

// Whole intervals are decoded in passes that share the memory of their
// destuffed bytes: a pass takes the intervals [iv0, iv0 + n_iv) of the list,
// their tiles and items.  Split intervals are destuffed with the pass that they
// lie in, to memory of their own, and decoded with the last.
struct GPass {
  uint32_t iv0, n_iv;
  uint32_t tile0, n_tiles;
  uint32_t item0, n_items;  // after the split intervals' items
};

// Device tables of a batch (one allocation).
struct GPlan {
  const GJob* jobs;
  const GInterval* ivs;
  const GTile* tiles;
  const GSplit* splits;
  const GGroup* groups;
  const uint32_t* split_of;  // per chunk
  const GItem* items;
  const uint32_t* skip_jobs;  // the jobs that have split intervals
  uint32_t n_skip;
  uint32_t many;  // entropy_follow's shape
  uint32_t n_iv, n_tiles, n_groups, n_more_groups, n_splits, n_long, n_items, n_split_items;
  GPass pass;
  uint8_t* data;      // destuffed bytes
  uint32_t* bytes;    // destuffed bytes per interval
  uint32_t* kept;     // per tile: bytes kept, bit 31 where the data ends in it
  uint32_t* status;   // per interval
  uint32_t* states;   // kSlots per chunk
  uint8_t* links;     // kSlots per chunk
  GHop* hops;         // kParts per slot
  GTask* tasks;       // kParts per chunk
  unsigned* counters;  // two of each decoding kernel's queue, and kMended
};

// A scan's tables into `codes` and `fast`, kTableSlots each.
static int tables_for(const mjd_scan& scan, GCodes* codes, FastTable* fast, uint32_t* tsel) {
  uint32_t used = 0;
  const int rc = plan_slots(scan, tsel, [&](int slot, const mjd_huffman& h, bool ac) {
    const int e = build_codes(h, &codes[slot]);
    if (e != kTableOk) return e;
    used |= 1u << slot;
    build_fast_table(codes[slot], ac, &fast[slot]);
    return e;
  });
  for (int i = 0; i < kTableSlots; ++i)
    if (!(used >> i & 1u)) {  // no code begins with anything
      memset(&codes[i], 0, sizeof(GCodes));
      build_fast_table(codes[i], false, &fast[i]);
    }
  switch (rc) {
    case kTableOk:
      return MJD_OK;
    case kTableUndefined:
      return fail(MJD_ECORRUPT, "scan uses an undefined Huffman table");
    case kTableTooMany:
      return fail(MJD_ECORRUPT, "Huffman table with more than 256 symbols");
    case kPlanTooManyTables:
      return fail(MJD_EUNSUPPORTED, "scan uses more than %d distinct Huffman tables (baseline uses at most 4); "
                                    "decode it on the host", kTableSlots);
    default:
      return fail(MJD_ECORRUPT, "Huffman code lengths overfill the code space");
  }
}

typedef __attribute__((address_space(3))) uint8_t lds8;
typedef __attribute__((address_space(3))) uint16_t lds16;
typedef __attribute__((address_space(3))) int16_t ldsi16;
typedef __attribute__((address_space(3))) uint32_t lds32;
typedef __attribute__((address_space(3))) uint64_t lds64;
typedef int v4i_t __attribute__((ext_vector_type(4)));
typedef uint32_t v4u_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) v4i_t lds128;
typedef __attribute__((address_space(1))) const uint8_t gin8;
typedef __attribute__((address_space(1))) const uint16_t gin16;
typedef __attribute__((address_space(1))) const v4u_t gin128;
typedef __attribute__((address_space(1))) v4i_t gout128;
typedef __attribute__((address_space(1))) uint8_t gout8;
typedef __attribute__((address_space(1), aligned(1))) uint32_t gout32u;  // any byte address
typedef uint32_t v4u_any __attribute__((ext_vector_type(4), aligned(1)));
typedef __attribute__((address_space(1))) v4u_any gout128u;

__device__ __forceinline__ uint32_t uniform(uint32_t v) {
  return static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(v)));
}
__device__ __forceinline__ uint32_t swap_bytes(uint32_t v) { return __builtin_amdgcn_perm(0, v, 0x00010203u); }
__device__ __forceinline__ uint32_t lane_of() { return threadIdx.x & 63u; }
// Lanes of `mask` below this one.
__device__ __forceinline__ uint32_t lanes_below(uint64_t mask) {
  return __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(mask >> 32),
                                   __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(mask), 0u));
}

// Makes a wave's LDS stores visible to its other lanes.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---- destuffing -----------------------------------------------------------------
// The zero that follows each 0xFF of a scan is dropped into a copy of the
// interval, so that the decoding lanes, which then take plain words, neither
// test every byte nor run the byte-wise path that one lane in six of a wave
// needs in every step.  One wave takes kTile raw bytes, 16 a lane, and leaves
// them by 16-byte stores at any address; bound by memory (15 us for the 17 MB
// of the 12-image corpus, of 322).  Data ends at the first 0xFF that no zero
// follows, as at the interval's end.

// Bits 0..3: the bytes of x that are zero.
__device__ __forceinline__ uint32_t zero_bytes(uint32_t x) {
  const uint32_t t = ~(((x & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | x | 0x7F7F7F7Fu);  // 0x80 in each zero byte
  return ((t >> 7) * 0x10204080u) >> 28 & 15u;
}

// Walks tile [a, b) of interval [start, end) of jpg; returns the bytes kept
// and whether the data ends in it.  STORE: also writes them from dst on.
template <bool STORE>
__device__ __forceinline__ uint32_t destuff_tile(gin8* jpg, uint32_t start, uint32_t end, uint32_t a, uint32_t b,
                                                 gout8* dst, bool* ends) {
  const uint32_t lane = lane_of();
  uint32_t total = 0;
  *ends = false;
  uint32_t p0 = a & ~15u;
  for (uint32_t left = b - p0;; left -= 1024, p0 += 1024) {  // counts down: b may lie within 1024 bytes of 2^32
    v4u_t v = {0, 0, 0, 0};
    uint32_t prev_ff = 0, next_zero = 0, in_iv = 0, in_tile = 0;
    if (16 * lane < left) {
      const uint32_t p = p0 + 16 * lane;
      v = *reinterpret_cast<gin128*>(jpg + p);
      if (p > start) prev_ff = jpg[p - 1] == 0xFFu;
      if (end - p > 16) next_zero = jpg[p + 16] == 0;
      const uint32_t lo_i = p < start ? start - p : 0, hi_i = end - p < 16 ? end - p : 16;
      const uint32_t lo_t = p < a ? a - p : 0, hi_t = b - p < 16 ? b - p : 16;
      in_iv = ((1u << hi_i) - 1u) & ~((1u << lo_i) - 1u);
      in_tile = ((1u << hi_t) - 1u) & ~((1u << lo_t) - 1u);
    }
    uint32_t ff = 0, zero = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      ff |= zero_bytes(~v[i]) << (4 * i);
      zero |= zero_bytes(v[i]) << (4 * i);
    }
    ff &= in_iv;
    zero &= in_iv;
    const uint32_t stop = ff & ~(zero >> 1 | next_zero << 15) & in_tile;
    uint32_t keep = in_tile & ~(zero & (ff << 1 | prev_ff));
    const uint64_t stops = __ballot(stop != 0);
    if (stops) {
      const uint32_t first = static_cast<uint32_t>(__builtin_ctzll(stops));
      keep = lane < first ? keep : (lane == first ? keep & ((stop & (0u - stop)) - 1u) : 0u);
    }
    const uint32_t n = static_cast<uint32_t>(__builtin_popcount(keep));
    uint32_t before = 0, all = 0;  // kept by the lanes below, and by the wave
#pragma unroll
    for (int i = 0; i < 5; ++i) {
      const uint64_t m = __ballot((n >> i & 1u) != 0);
      before += lanes_below(m) << i;
      all += static_cast<uint32_t>(__builtin_popcountll(m)) << i;
    }
    if constexpr (STORE) {
      gout8* to = dst + total + before;
      if (keep == 0xFFFFu) {
        *reinterpret_cast<gout128u*>(to) = v;
      } else if (keep) {
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (keep >> i & 1u) *to++ = static_cast<uint8_t>(v[i >> 2] >> (8 * (i & 3)));
      }
    }
    total += all;
    *ends = stops != 0;
    if (stops || left <= 1024) return total;
  }
}

__global__ __launch_bounds__(kThreads) void entropy_destuff_count(const GPlan pl) {
  const uint32_t w = uniform(blockIdx.x * kWaves + (threadIdx.x >> 6));
  if (w >= pl.pass.n_tiles) return;
  const GTile t = pl.tiles[pl.pass.tile0 + w];
  const GInterval iv = pl.ivs[t.iv];
  const uint32_t a = iv.start + t.index * kTile;
  const uint32_t b = iv.end - a < kTile ? iv.end : a + kTile;
  bool ends;
  const uint32_t n = destuff_tile<false>((gin8*)pl.jobs[iv.job].jpg, iv.start, iv.end, a, b, nullptr, &ends);
  if (lane_of() == 0) pl.kept[pl.pass.tile0 + w] = n | (ends ? 0x80000000u : 0u);
}

// One entry per lane of a job's skip tables.
__device__ __forceinline__ void fill_skip_tables(const GPlan& pl, uint32_t i) {
  constexpr uint32_t kAll = kTableSlots * kSkipEntries;
  if (i >= pl.n_skip * kAll) return;
  const GJob& jb = pl.jobs[pl.skip_jobs[i / kAll]];
  const uint32_t at = i % kAll, t = at / kSkipEntries;
  bool ac = false;
  for (uint32_t b = 0; b < jb.bpm; ++b) ac = ac || (jb.ac_slots >> (2 * b) & 3u) == t;
  const FastTable& ft = jb.tables->t[t];
  jb.skip[at] = static_cast<uint16_t>(skip_entry(at % kSkipEntries, ac, [&](uint32_t top) {
    const uint32_t e = ft.fast[top >> (32 - kGLook)];
    return e & 31u ? e : more_entry(e, top, ac, [&](uint32_t k) { return static_cast<uint32_t>(ft.more[k]); },
                                    CodeTab{jb.codes}, static_cast<int>(t));
  }));
}

// One wave per interval of at most kTile bytes, then one per tile of the
// longer ones, after the bytes that entropy_destuff_count found in the tiles before;
// the workgroups after those fill the skip tables that entropy_guess and
// entropy_follow read.
__global__ __launch_bounds__(kThreads) void entropy_destuff(const GPlan pl) {
  const GPass ps = pl.pass;
  const uint32_t groups = (ps.n_iv + ps.n_tiles + kWaves - 1) / kWaves;
  if (blockIdx.x >= groups) return fill_skip_tables(pl, (blockIdx.x - groups) * kThreads + threadIdx.x);
  const uint32_t w = uniform(blockIdx.x * kWaves + (threadIdx.x >> 6));
  if (w >= ps.n_iv + ps.n_tiles) return;
  const uint32_t lane = lane_of();
  uint32_t which = ps.iv0 + w, tile = 0, at = 0;
  if (w >= ps.n_iv) {
    const GTile t = pl.tiles[ps.tile0 + w - ps.n_iv];
    which = t.iv;
    tile = t.index;
    bool ended = false;
    for (uint32_t i = lane; i < tile; i += 64) {
      const uint32_t k = pl.kept[ps.tile0 + t.first + i];
      at += k & 0x7FFFFFFFu;
      ended = ended || (k >> 31);
    }
    for (int d = 32; d; d >>= 1) at += static_cast<uint32_t>(__shfl_xor(static_cast<int>(at), d));
    at = uniform(at);
    if (__ballot(ended)) return;
  }
  const GInterval iv = pl.ivs[which];
  if (w < ps.n_iv) {
    if (lane == 0) pl.status[which] = kStatusOk;
    if (lane == 0 && which == 0) pl.counters[kMended] = 0;
    if (iv.end - iv.start > kTile) return;
  }
  const uint32_t a = iv.start + tile * kTile;
  const uint32_t b = iv.end - a < kTile ? iv.end : a + kTile;
  gout8* dst = (gout8*)(pl.data + static_cast<uint64_t>(iv.dst) * 16);
  bool ends;
  at += destuff_tile<true>((gin8*)pl.jobs[iv.job].jpg, iv.start, iv.end, a, b, dst + at, &ends);
  if (ends || b == iv.end) {  // zeros up to the end of the chunk after the last
    if (lane == 0) pl.bytes[which] = at;
    if (lane < 8) *reinterpret_cast<gout32u*>(dst + at + 4 * lane) = 0;
  }
}

// ---- tables and words in LDS -------------------------------------------------------

typedef __attribute__((address_space(3))) FastTables lds_tables;

// By all lanes of a workgroup.
template <uint32_t THREADS>
__device__ __forceinline__ void load_tables(const FastTables* from, lds_tables* to) {
  gin128* src = (gin128*)from;
  __attribute__((address_space(3))) v4u_t* dst = (__attribute__((address_space(3))) v4u_t*)to;
  for (uint32_t i = threadIdx.x; i < sizeof(FastTables) / 16; i += THREADS) dst[i] = src[i];
}

// The `fast` entry at the front of `top` in the table at byte offset t, and
// the whole one where that uses no bits.
__device__ __forceinline__ uint32_t fast_entry(const lds_tables* tabs, uint32_t t, uint32_t top) {
  return *reinterpret_cast<const lds16*>((const lds8*)tabs + t + (top >> 21 & 0x7FEu));
}
__device__ __forceinline__ uint32_t long_code(const lds_tables* tabs, const GCodes* codes, uint32_t t, uint32_t top,
                                              uint32_t e, bool ac) {
  const lds16* more = reinterpret_cast<const lds16*>((const lds8*)tabs + t + sizeof(FastTable::fast));
  return more_entry(e, top, ac, [more](uint32_t i) { return static_cast<uint32_t>(more[i]); }, CodeTab{codes},
                    static_cast<int>(t / sizeof(FastTable)));
}
// Byte offset of the table that two bits of `slots` name for block b.
__device__ __forceinline__ uint32_t table_of(uint32_t slots, uint32_t b) {
  return (slots >> (2 * b) & 3u) * static_cast<uint32_t>(sizeof(FastTable));
}

// Words of consecutive chunks, which a workgroup copies to LDS before it
// walks through them: a lane then waits for no load.  A lane's words are
// counted from the start of its interval and end with a zero word past the
// data.
// Words that a block needs past the word of its first bit, the window's
// included: a DC symbol of at most 27 bits and 63 of at most 31.
constexpr uint32_t kBlockWords = (63 * 31 + 27 + 31) / 32 + 2;

// Copies n words (a multiple of 4) from `src` on, by `lanes` lanes.
__device__ __forceinline__ void stage_words(lds32* base, gin128* src, uint32_t n, uint32_t lane, uint32_t lanes) {
  for (uint32_t i = lane; i < n / 4; i += lanes) {
    const v4u_t v = src[i];
#pragma unroll
    for (uint32_t j = 0; j < 4; ++j) base[4 * i + j] = swap_bytes(v[j]);
  }
}

struct StagedWords {
  lds32* base;
  gin128* src;    // the interval's data
  uint32_t off;   // place of its first word in the copy (modulo 2^32)
  uint32_t n;     // words of the copy
  uint32_t zero;  // its zero word

  __device__ uint32_t word(uint32_t w) const {
    const uint32_t v = w < zero ? w : zero, i = v + off;
    if (__builtin_expect(i < n, 1)) return base[i];
    return swap_bytes(((__attribute__((address_space(1))) const uint32_t*)src)[v]);
  }
  __device__ BitWindow open(uint32_t at, uint32_t bit) const {
    const uint32_t q = window_word(at, bit);
    return window_at(at, bit, word(q ? q - 1 : 0), word(q));
  }
};

// Eight words per lane in LDS (word w at [w & 7][lane], so that lanes at
// different words meet no bank twice), filled from 16-byte chunks.  A chunk
// is loaded at one refill and put in place at the next, so its latency
// passes while the lane decodes; chunks past the data are the zero chunk
// that destuffing leaves there.
constexpr uint32_t kRingWords = 8;
struct WordRing {
  lds32* base;
  gin128* src;
  uint32_t last;  // the zero chunk
  uint32_t have;  // words below are in place
  v4u_t chunk;
  bool loading;

  __device__ void put(uint32_t at, v4u_t c) {
#pragma unroll
    for (uint32_t i = 0; i < 4; ++i) base[((at & 4u) + i) * kThreads] = swap_bytes(c[i]);  // at: a multiple of 4
  }
  __device__ uint32_t word(uint32_t w) const { return base[(w & (kRingWords - 1)) * kThreads]; }
  // A window at bit 32 * word + bit of `bytes` bytes.
  __device__ BitWindow open(uint32_t bytes, uint32_t word_, uint32_t bit) {
    last = bytes / 16 + 1;  // there is always the zero chunk
    const uint32_t c = word_ / 4 < last ? word_ / 4 : last;
    const v4u_t c0 = src[c], c1 = src[c < last ? c + 1 : last];
    have = 4 * (word_ / 4);
    put(have, c0);
    put(have + 4, c1);
    have += 8;
    loading = false;
    const uint32_t q = window_word(word_, bit);
    return window_at(word_, bit, word(q - 1), word(q));
  }
  __device__ void refill(bool active, uint32_t wi) {
    if (loading) {
      put(have, chunk);
      have += 4;
    }
    loading = active && have - (wi & ~3u) <= 4;
    if (loading) chunk = src[(have >> 2) < last ? have >> 2 : last];
  }
  __device__ bool ready(uint32_t wi) const { return wi < have; }
};

// ---- finding the block boundaries of a split interval -----------------------------
// A Huffman-coded stream read from a wrong bit falls into step with the code
// words within a few tens of bytes, but its blocks may then be counted in the
// wrong place of the MCU, and the tables of luma and chroma differ, so the
// step is lost and found again until the place is right too: about 130 bytes
// on average for 4:2:0, over 500 for one start in a hundred.  With one lane
// per possible first block, one of them is right within 20 bytes for 19
// starts of 20 (measured over qualities 50 to 95).
//   guess    one lane per chunk and first block reads the chunk from its first
//            bit and leaves the block boundary at which it enters the next;
//   follow   one lane per distinct boundary reads on through that chunk,
//            counts blocks and sums DC differences, and links the boundary to
//            the one of the next chunk that it arrives at.  A lane that
//            arrives elsewhere takes a free slot there and goes on;
//   resolve  chains the links from the interval's start (a scan over maps of
//            slots), and turns counts and sums into each chunk's task.
// A chain breaks where the boundary it arrives at has no slot (none was free,
// or the lane had gone on for kMaxHops chunks): dense blocks, whose lanes take
// long to fall into step, and content that repeats.  entropy_resolve then lets
// one lane read on to the next boundary that has been followed, and scans
// again.  The exits that a guess repeats leave their slots free, which makes
// breaks rare up to quality 90 (none in 64 files of quality 50 and 85).  Noisy
// 1024x768 files without markers have 13 at quality 95 and 500 to 750 at 98,
// and take 0.6 and 17 to 27 ms; 100 and 155 when one lane decoded the rest of
// the interval instead.
// Both kernels are bound by a lane's chain of look-ups where lanes are few and
// by instruction issue where they are many, so a look-up takes several symbols
// (skip tables; 11 bits of look-up instead of 12 cost 2% and leave room for
// four workgroups a CU), and what only a block's end needs is done once in
// kLooks look-ups, for the lanes that have come to one: a 4000x3000 4:2:0 file
// with a marker per MCU row takes 31 + 55 us in them, the 12-image corpus 90 +
// 77 us (48 + 75 and 115 + 110 with an end in every look-up).
constexpr uint32_t kMaxHops = 32;

// The skip tables of a job in LDS, and its whole tables, which one lane in
// 300 needs in a step: in LDS too, or in memory, which leaves room for half
// as many waves again.
template <bool WHOLE>
struct SkipLds {
  __align__(16) uint16_t skip[kTableSlots * kSkipEntries];
  __align__(16) FastTables fast[WHOLE ? 1 : 0];
};

template <bool WHOLE, uint32_t THREADS>
__device__ __forceinline__ void load_skip_tables(const GJob& jb, SkipLds<WHOLE>* to) {
  if constexpr (WHOLE) load_tables<THREADS>(jb.tables, (lds_tables*)&to->fast[0]);
  gin128* src = (gin128*)jb.skip;
  __attribute__((address_space(3))) v4u_t* dst = (__attribute__((address_space(3))) v4u_t*)to->skip;
  for (uint32_t i = threadIdx.x; i < kTableSlots * kSkipEntries / 8; i += THREADS) dst[i] = src[i];
}

// A lane on its way from a block boundary to another, over a copy of the
// data.  A step's instructions are what it costs (a wave alone on its SIMD
// issues one in five cycles, and a look-up's latency is that of twenty-five),
// so whatever only a block's end needs waits for one: the position, the next
// block's tables, the sum that its DC difference goes to.  Of a wave's 64
// lanes some end a block in nearly every look-up, so up to kLooks look-ups are
// made first, by the lanes that have not come to an end (2: 182, 3: 168, 4:
// 168, 5: 167 us for the file with markers per row, 345, 324, 325 and 327 for
// the corpus); a block's DC symbol is then always in the first of them.
constexpr int kLooks = 4;
template <bool WHOLE, uint32_t THREADS>
struct Walker {
  const lds16* skip;
  const lds_tables* fast;    // WHOLE
  const FastTables* memory;  // else
  const GCodes* codes;
  uint32_t bpm2, slots_dc, slots_ac, comp_bits;
  uint32_t w0, w1;  // the window, as in BitWindow
  int32_t sh;
  uint32_t at;      // byte offset in the copy of the word after w1's
  uint32_t b2, k;   // twice the block of the MCU; the zig-zag position
  uint32_t t, ac;   // slots of the next symbol's table and of the block's AC table
  lds32* sums;      // of DC differences, a row of THREADS lanes for each component
  uint32_t row;     // byte offset of the block's
  uint32_t blocks;

  __device__ Walker(const GJob& jb, const SkipLds<WHOLE>* tabs, lds32* sums_)
      : skip((const lds16*)tabs->skip), fast((const lds_tables*)tabs->fast), memory(jb.tables), codes(jb.codes), bpm2(2 * jb.bpm), slots_dc(jb.dc_slots), slots_ac(jb.ac_slots),
        comp_bits(jb.comp_bits), sums(sums_), blocks(0) {}
  // The lane's window, from one over words counted from `off` words into the copy.
  __device__ void open(const BitWindow& w, uint32_t off) {
    w0 = w.w0;
    w1 = w.w1;
    sh = w.sh;
    at = 4 * (w.wi + off);
  }
  __device__ void block(uint32_t b2_) {
    b2 = b2_;
    k = 0;
    t = slots_dc >> b2 & 3u;
    ac = slots_ac >> b2 & 3u;
    row = (comp_bits >> b2 & 3u) * (THREADS * 4);
  }
  // The entry of the code at the front of `top` in the table of slot s.
  __device__ uint32_t whole_entry(uint32_t s, uint32_t top) const {
    if constexpr (WHOLE) {
      const uint32_t ft = s * static_cast<uint32_t>(sizeof(FastTable)), e = fast_entry(fast, ft, top);
      return e & 31u ? e : long_code(fast, codes, ft, top, e, k != 0);
    } else {
      const FastTable& ft = memory->t[s];
      const uint32_t e = ft.fast[top >> (32 - kGLook)];
      return e & 31u ? e : more_entry(e, top, k != 0, [&](uint32_t i) { return static_cast<uint32_t>(ft.more[i]); },
                                      CodeTab{codes}, static_cast<int>(s));
    }
  }
  // Position of the next unread bit in the copy, modulo 2^32.
  __device__ uint32_t pos() const { return 8 * at - 32u - static_cast<uint32_t>(sh); }
  // Walks on from a block boundary until ended(its position) at one; next(at)
  // reads the word at a byte offset.  Where no code begins, the block ends
  // (the decoding lane will find the error in it) and the lane goes on a bit
  // later with a new first block.
  template <bool COUNT, class Next, class Ended>
  __device__ __forceinline__ void walk(const Next& next, const Ended& ended) {
    const auto add_dc = [&](uint32_t top, uint32_t bits, uint32_t size) {
      __hip_atomic_fetch_add(reinterpret_cast<lds32*>(reinterpret_cast<lds8*>(sums) + row),
                             static_cast<uint32_t>(entry_value(top, bits, size)), __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_WAVEFRONT);
    };
    const auto drop = [&](uint32_t bits, uint32_t word) {
      sh -= static_cast<int32_t>(bits);
      const bool over = sh < 0;
      sh &= 31;
      w0 = over ? w1 : w0;
      w1 = over ? word : w1;
      at += over ? 4u : 0u;
    };
    uint32_t top, m, word, bits, to;
    const auto look = [&]() {
      top = __builtin_amdgcn_alignbit(w0, w1, static_cast<uint32_t>(sh));
      m = skip[__builtin_amdgcn_alignbit(t, top, 32 - kSkipLook)];
      word = next(at);
      bits = m & 31u;
      to = k + (m >> 5 & 127u);
    };
    for (bool on = true; on;) {
      look();
#pragma unroll
      for (int i = 1; i < kLooks; ++i) {
        if (to > 63) break;
        if (COUNT && i == 1) add_dc(top, bits, m >> 12);  // 0 for AC symbols
        k = to;
        t = ac;
        drop(bits, word);
        look();
      }
      t = ac;
      bool ends = to > 63;
      if (ends) {
        bool bad = false;
        if (skip_takes_one(m, to)) {
          const uint32_t e = whole_entry(k ? ac : slots_dc >> b2 & 3u, top);
          bad = e == kBadEntry;
          bits = bad ? 1u : e & 31u;
          if (COUNT && k == 0 && !bad) add_dc(top, bits, e >> 5 & 15u);
          to = k + (e >> 9);
          ends = to > 63;
        }
        if (ends) {
          if constexpr (COUNT) ++blocks;
          block(bad || b2 + 2 == bpm2 ? 0u : b2 + 2);
          to = 0;
          on = !ended(pos() + bits);
        }
      }
      k = to;
      drop(bits, word);
    }
  }
};

// Words that a workgroup stages of its chunks and those after them, for a
// block that begins in the last chunk and, in `follow`, for lanes that go on.
// A lane per guess: 85 chunks of six blocks an MCU.  512 lanes to a copy of
// the tables, as 256 left half as many waves a CU (145 us in entropy_guess for
// the 12-image corpus, 115 here).
constexpr uint32_t kGuessThreads = 512, kGuessGroup = 85;
constexpr uint32_t kGuessWords = (kGuessGroup * kChunkWords + kBlockWords + 3) & ~3u;
// About two boundaries a chunk to follow.  Where more chunks come together
// than the small workgroups hold that fit on the chip at once, larger ones
// with the whole tables in memory have twice the waves a CU: 145 -> 110 us for
// the corpus (133,000 chunks); with 19,500 chunks and with 4,000 the small
// ones take 76 and 65 us, the large ones 81 and 70.
template <bool MANY>
struct FollowShape {
  static constexpr uint32_t THREADS = MANY ? 512 : 256, GROUP = MANY ? 208 : 96, MORE = 8;  // chunks
  static constexpr uint32_t WORDS = (GROUP + MORE) * kChunkWords;
  static constexpr uint32_t RESIDENT = 3;  // workgroups a CU
};

// A lane's chunk: its interval, its number there and the last one that holds
// data, which hands over to none.
struct ChunkOf {
  GSplit sp;
  uint32_t c, last;
  StagedWords words;
  uint32_t limit;  // byte offset of the zero word in the copy
  __device__ ChunkOf(const GPlan& pl, const GGroup& g, uint32_t chunk, lds32* staged, uint32_t n) {
    sp = pl.splits[pl.split_of[chunk]];
    c = chunk - sp.chunk0;
    const uint32_t bytes = pl.bytes[sp.iv];
    last = bytes ? (bytes - 1) / kChunk : 0;
    words.base = staged;
    words.src = (gin128*)(pl.data + static_cast<uint64_t>(sp.chunk0) * kChunk);
    words.off = (sp.chunk0 - g.first) * kChunkWords;
    words.n = n;
    words.zero = (bytes + 3) / 4;
    limit = 4 * (words.zero + words.off);
  }
  // A word that is known to lie in the copy, or past the data.
  __device__ uint32_t staged(uint32_t at) const {
    return *reinterpret_cast<const lds32*>(reinterpret_cast<const lds8*>(words.base) + (at < limit ? at : limit));
  }
};

__global__ __launch_bounds__(kGuessThreads) void entropy_guess(const GPlan pl) {
  __shared__ SkipLds<true> tables;
  __shared__ uint32_t staged[kGuessWords];
  __shared__ uint32_t exits[kGuessThreads];
  const GGroup g = pl.groups[blockIdx.x];
  const GJob& jb = pl.jobs[g.job];
  const uint32_t n = (g.count * kChunkWords + kBlockWords + 3) & ~3u;
  stage_words((lds32*)staged, (gin128*)(pl.data + static_cast<uint64_t>(g.first) * kChunk), n, threadIdx.x, kGuessThreads);
  load_skip_tables<true, kGuessThreads>(jb, &tables);
  __syncthreads();
  Walker<true, kGuessThreads> walk(jb, &tables, nullptr);
  const uint32_t tries = jb.bpm, mine = threadIdx.x / tries, first = threadIdx.x - mine * tries;
  const bool used = mine < g.count;
  const uint32_t chunk = g.first + (used ? mine : 0u);
  const ChunkOf at(pl, g, chunk, (lds32*)staged, n);
  uint32_t state = kNoState;
  if (used && at.c < at.last && (at.c > 0 || first == 0)) {
    const uint32_t target = (mine + 1) * (kChunk * 8);
    walk.open(at.words.open(at.c * kChunkWords, 0), at.words.off);
    walk.block(2 * first);
    walk.walk<false>([&](uint32_t i) { return at.staged(i); },
                     [&](uint32_t pos) { return static_cast<int32_t>(pos - target) >= 0; });
    state = make_state(walk.pos() - target, walk.b2 / 2) | kGuessed;
  }
  exits[threadIdx.x] = state;
  __syncthreads();
  if (!used) return;
  for (uint32_t j = 0; j < first; ++j)
    if (exits[threadIdx.x - first + j] == state) state = kNoState;
  uint32_t* own = pl.states + static_cast<uint64_t>(chunk) * kSlots;
  if (at.c == 0 && first == 0) {
    own[0] = make_state(0, 0) | kGuessed;
    for (uint32_t i = 1; i < kSlots; ++i) own[i] = kNoState;
  }
  if (at.c + 1 < at.sp.n_chunks) {
    own[kSlots + first] = state;
    if (first == 0)
      for (uint32_t i = tries; i < kSlots; ++i) own[kSlots + i] = kNoState;
  }
}

template <bool MANY>
__global__ __launch_bounds__(FollowShape<MANY>::THREADS) void entropy_follow(const GPlan pl) {
  using F = FollowShape<MANY>;
  constexpr uint32_t THREADS = F::THREADS;
  __shared__ SkipLds<!MANY> tables;
  __shared__ uint32_t staged[F::WORDS];
  __shared__ uint32_t sums[3 * THREADS];
  __shared__ uint16_t list[F::GROUP * kGuesses];  // chunk in the group << 3 | slot of the boundaries that were guessed
  __shared__ uint32_t n_list;
  const GGroup g = pl.groups[pl.n_groups + blockIdx.x];
  const GJob& jb = pl.jobs[g.job];
  const uint32_t n = (g.count + F::MORE) * kChunkWords;
  if (threadIdx.x == 0) n_list = 0;
  stage_words((lds32*)staged, (gin128*)(pl.data + static_cast<uint64_t>(g.first) * kChunk), n, threadIdx.x, THREADS);
  load_skip_tables<!MANY, THREADS>(jb, &tables);
  __syncthreads();
  Walker<!MANY, THREADS> walk(jb, &tables, (lds32*)sums + threadIdx.x);
  const uint32_t tries = jb.bpm;
  for (uint32_t i0 = 0; i0 < g.count * tries; i0 += THREADS) {
    const uint32_t i = i0 + threadIdx.x, mine = i / tries, slot = i - mine * tries;
    bool use = mine < g.count;
    if (use) {
      // not those that a lane of the chunk before has put there by now
      const uint32_t own = pl.states[static_cast<uint64_t>(g.first + mine) * kSlots + slot];
      use = own != kNoState && (own & kGuessed);
    }
    const uint64_t m = __ballot(use);
    uint32_t base = 0;
    if (lane_of() == 0) base = atomicAdd(&n_list, static_cast<uint32_t>(__builtin_popcountll(m)));
    base = uniform(base);
    if (use) list[base + lanes_below(m)] = static_cast<uint16_t>(mine << 3 | slot);
  }
  __syncthreads();
  const uint32_t n_work = n_list;
  for (uint32_t i = threadIdx.x; i < n_work; i += THREADS) {
    uint32_t chunk = g.first + (list[i] >> 3), slot = list[i] & 7u, hops = 0;
    const ChunkOf at(pl, g, chunk, (lds32*)staged, n);
    uint32_t c = at.c;
    if (c >= at.last) continue;
    const uint32_t from = pl.states[static_cast<uint64_t>(chunk) * kSlots + slot] & ~kGuessed;
    walk.open(at.words.open(c * kChunkWords + (from >> 8), (from >> 3) & 31u), at.words.off);
    walk.block(2 * (from & 7u));
    for (bool on = true; on;) {
      uint32_t* to = pl.states + static_cast<uint64_t>(chunk + 1) * kSlots;
      uint32_t guessed[kGuesses];  // asked for before the walk
      for (uint32_t j = 0; j < kGuesses; ++j) guessed[j] = to[j];
      const bool in_copy = (chunk + 1 - g.first) * kChunkWords + kBlockWords <= n;
      // The parts' ends in the copy: the first leaves what was counted up to
      // it and the lane goes on to the second, unless its block goes past both.
      const uint32_t end0 = (chunk - g.first) * (kChunk * 8) + kPart * 8, end1 = end0 + kPart * 8;
      uint32_t state0 = kNoState, blocks0 = 0, sum0[3] = {0, 0, 0};
      lds32* sum = (lds32*)sums + threadIdx.x;
      for (uint32_t d = 0; d < 3; ++d) sum[d * THREADS] = 0;
      walk.blocks = 0;
      const auto ended = [&](uint32_t pos) {
        if (static_cast<int32_t>(pos - end0) < 0) return false;
        if (state0 == kNoState) {
          state0 = make_state(pos - end0, walk.b2 / 2);
          blocks0 = walk.blocks;
          for (uint32_t d = 0; d < 3; ++d) sum0[d] = sum[d * THREADS];
        }
        return static_cast<int32_t>(pos - end1) >= 0;
      };
      if (!ended(walk.pos())) {
        if (in_copy) walk.template walk<true>([&](uint32_t i) { return at.staged(i); }, ended);
        else walk.template walk<true>([&](uint32_t i) { return at.words.word(i / 4 - at.words.off); }, ended);
      }
      const uint32_t state = make_state(walk.pos() - end1, walk.b2 / 2);
      GHop* hop = pl.hops + (static_cast<uint64_t>(chunk) * kSlots + slot) * kParts;
      GHop h0{static_cast<uint16_t>(blocks0), {}, state0, 0}, h1{static_cast<uint16_t>(walk.blocks - blocks0), {}, state, 0};
      for (uint32_t d = 0; d < 3; ++d) {
        h0.dc[d] = static_cast<uint16_t>(sum0[d]);
        h1.dc[d] = static_cast<uint16_t>(sum[d * THREADS] - sum0[d]);
      }
      hop[0] = h0;
      hop[1] = h1;
      uint32_t link = kNoLink;
      for (uint32_t j = kGuesses; j-- > 0;)
        if (guessed[j] == (state | kGuessed)) link = j;
      on = false;  // unless this lane goes on from a slot of its own
      if (link == kNoLink && ++hops < kMaxHops) {
        // the first free slot; whoever took it for the same boundary before
        // found those below it taken too
#pragma unroll
        for (uint32_t j = 0; j < kSlots; ++j) {
          if (link != kNoLink || (j < kGuesses && guessed[j] != kNoState && (guessed[j] & kGuessed))) continue;
          const uint32_t was = atomicCAS(&to[j], kNoState, state);
          if (was == kNoState || was == state) link = j;
          on = was == kNoState;
        }
      }
      pl.links[static_cast<uint64_t>(chunk) * kSlots + slot] = static_cast<uint8_t>(link);
      on = on && c + 1 < at.last;
      ++c;
      ++chunk;
      slot = link;
    }
  }
}

// Scans rows of N words over a group of LANES lanes (64: a wave; more: the
// workgroup): what then() makes of those of all lanes below goes to `below`,
// of the whole group's to `all`.
template <int LANES, int N, class Then>
__device__ __forceinline__ void scan(const uint32_t (&v)[N], const uint32_t (&none)[N], Then then, uint32_t* lds,
                                     uint32_t (&below)[N], uint32_t (&all)[N]) {
  const uint32_t lane = lane_of();
  const auto wave_scan = [&](uint32_t (&x)[N], uint32_t width) {
    for (uint32_t d = 1; d < width; d <<= 1) {
      uint32_t y[N];
#pragma unroll
      for (int i = 0; i < N; ++i) y[i] = static_cast<uint32_t>(__shfl_up(static_cast<int>(x[i]), d));
      then(y, x);  // y: the result
#pragma unroll
      for (int i = 0; i < N; ++i) x[i] = lane >= d ? y[i] : x[i];
    }
  };
  uint32_t x[N];
  for (int i = 0; i < N; ++i) x[i] = v[i];
  wave_scan(x, 64);
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const uint32_t y = static_cast<uint32_t>(__shfl_up(static_cast<int>(x[i]), 1));
    below[i] = lane ? y : none[i];
    all[i] = static_cast<uint32_t>(__shfl(static_cast<int>(x[i]), 63));
  }
  if constexpr (LANES > 64) {
    constexpr uint32_t kGroupWaves = LANES / 64;
    const uint32_t wave = uniform(threadIdx.x >> 6);
    if (lane == 0)
      for (int i = 0; i < N; ++i) lds[i * kGroupWaves + wave] = all[i];
    __syncthreads();
    uint32_t y[N];  // each wave scans the waves' values
#pragma unroll
    for (int i = 0; i < N; ++i) y[i] = lds[i * kGroupWaves + lane % kGroupWaves];
    wave_scan(y, kGroupWaves);
    __syncthreads();
    uint32_t before[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
      before[i] = wave ? static_cast<uint32_t>(__shfl(static_cast<int>(y[i]), static_cast<int>(wave) - 1)) : none[i];
      all[i] = static_cast<uint32_t>(__shfl(static_cast<int>(y[i]), kGroupWaves - 1));
    }
    then(before, below);
#pragma unroll
    for (int i = 0; i < N; ++i) below[i] = before[i];
  }
}

// Reads on from a block boundary of chunk c of a split interval to the first
// one past it and leaves the hops of its parts; returns the boundary as a
// state of the next chunk.  One lane, its tables and words in memory: 128
// bytes take 22 us, most of them the latency of the look-ups (70 with one
// symbol a look-up, more than the 50 that entropy_decode needs for them, so
// content that never falls into step is read at no loss).
__device__ __forceinline__ uint32_t walk_chunk(const GPlan& pl, const GSplit& sp, const GJob& jb, uint32_t bytes,
                                               uint32_t c, uint32_t state, GHop* hops) {
  StagedWords words;
  words.base = nullptr;  // no copy
  words.src = (gin128*)(pl.data + static_cast<uint64_t>(sp.chunk0) * kChunk);
  words.off = words.n = 0;
  words.zero = (bytes + 3) / 4;
  const uint32_t bpm = jb.bpm, comp_bits = jb.comp_bits, slots_dc = jb.dc_slots, slots_ac = jb.ac_slots;
  gin16* skip = (gin16*)jb.skip;
  const CodeTab codes{jb.codes};
  BitWindow w = words.open(c * kChunkWords + (state >> 8), (state >> 3) & 31u);
  uint32_t pos = state >> 3, b = state & 7u;  // in bits of the chunk
#pragma unroll 1
  for (uint32_t j = 0; j < kParts; ++j) {
    const uint32_t end = (j + 1) * kPart * 8;
    uint32_t blocks = 0, d0 = 0, d1 = 0, d2 = 0;
    while (pos < end) {
      bool bad = false;
      uint32_t t = slots_dc >> (2 * b) & 3u, dc = 0;
      for (uint32_t k = 0; k < 64;) {
        const uint32_t top = w.top(), next = words.word(w.wi);
        const uint32_t m = skip[t * kSkipEntries + (top >> (32 - kSkipLook))];
        uint32_t bits = m & 31u, size = m >> 12, to = k + (m >> 5 & 127u);
        if (to > 63 && skip_takes_one(m, to)) {
          gin16* ft = (gin16*)jb.tables + t * (sizeof(FastTable) / 2);  // fast, then more
          uint32_t e = ft[top >> (32 - kGLook)];
          if ((e & 31u) == 0)
            e = more_entry(e, top, k != 0, [ft](uint32_t i) { return static_cast<uint32_t>(ft[(1u << kGLook) + i]); }, codes,
                           static_cast<int>(t));
          bad = e == kBadEntry;
          bits = bad ? 1u : e & 31u;
          size = bad ? 0u : e >> 5 & 15u;
          to = k + (e >> 9);
        }
        if (k == 0) dc = static_cast<uint32_t>(entry_value(top, bits, size));
        t = slots_ac >> (2 * b) & 3u;
        w.drop(bits, next);
        pos += bits;
        k = to;
      }
      const uint32_t comp = comp_bits >> (2 * b) & 3u;
      d0 += comp == 0 ? dc : 0u;
      d1 += comp == 1 ? dc : 0u;
      d2 += comp == 2 ? dc : 0u;
      ++blocks;
      b = bad || b + 1 == bpm ? 0u : b + 1;
    }
    hops[j] = GHop{static_cast<uint16_t>(blocks),
                   {static_cast<uint16_t>(d0), static_cast<uint16_t>(d1), static_cast<uint16_t>(d2)},
                   make_state(pos - end, b), 0};
  }
  return make_state(pos - kChunk * 8, b);
}

// Mends the chain of a split interval that ends at chunk c, entered by slot
// `slot`: the boundary it arrives at has no slot in chunk c + 1.  No slot of
// that chunk but this boundary's matters then, so it takes the first one, and
// the lane reads on until it arrives at a boundary that has been followed.
__device__ __forceinline__ void mend_chain(const GPlan& pl, const GSplit& sp, const GJob& jb, uint32_t bytes,
                                           uint32_t last, uint32_t c, uint32_t slot) {
  const auto at = [&](uint32_t chunk, uint32_t i) { return static_cast<uint64_t>(sp.chunk0 + chunk) * kSlots + i; };
  uint32_t state = pl.hops[at(c, slot) * kParts + kParts - 1].state;
  for (;;) {
    uint32_t link = kNoLink;
    for (uint32_t j = 0; j < kSlots; ++j) {
      const uint32_t there = pl.states[at(c + 1, j)];
      if (there != kNoState && (there & ~kGuessed) == state) link = j;
    }
    const bool met = link != kNoLink;
    pl.links[at(c, slot)] = static_cast<uint8_t>(met ? link : 0u);
    if (met) return;
    ++c;
    slot = 0;
    pl.states[at(c, 0)] = state;
    if (c == last) return;
    state = walk_chunk(pl, sp, jb, bytes, c, state, pl.hops + at(c, 0) * kParts);
  }
}

// One group of LANES lanes per split interval: a wave for most, a workgroup
// for those of many chunks (pl.n_long of them, first in the list).  A lane
// takes a run of chunks, kRun at a time so that their loads overlap.  Where
// waves resolve, five of them to a SIMD: the 9619 intervals of the 12-image
// corpus take 16.9 us, 19 with the 112 registers that mending asks for otherwise
// (16.4 without mending).
constexpr uint32_t kRun = 4;
template <int LANES>
__global__ __launch_bounds__(LANES > 64 ? LANES : kThreads, LANES > 64 ? 4 : 5) void entropy_resolve(const GPlan pl) {
  __shared__ uint32_t lds[LANES > 64 ? 4 * (LANES / 64) : 1];
  const uint32_t which = LANES > 64 ? blockIdx.x : pl.n_long + uniform(blockIdx.x * kWaves + (threadIdx.x >> 6));
  if (which >= pl.n_splits) return;
  const uint32_t id = LANES > 64 ? threadIdx.x : lane_of();
  const GSplit sp = pl.splits[which];
  const GInterval iv = pl.ivs[sp.iv];
  const GJob jb = pl.jobs[iv.job];
  const uint32_t bytes = pl.bytes[sp.iv];
  const uint32_t last = bytes ? (bytes - 1) / kChunk : 0;
  const uint32_t per = (last + LANES - 1) / LANES;
  const uint32_t c0 = id * per < last ? id * per : last, c1 = c0 + per < last ? c0 + per : last;
  const uint64_t* links = reinterpret_cast<const uint64_t*>(pl.links) + sp.chunk0;
  // the maps of a run of chunks from chunk c on
  auto load_maps = [&](uint32_t c, SlotMap (&maps)[kRun]) {
    uint64_t l[kRun];
#pragma unroll
    for (uint32_t i = 0; i < kRun; ++i) l[i] = links[c + i < c1 ? c + i : c];
#pragma unroll
    for (uint32_t i = 0; i < kRun; ++i) maps[i] = map_of_links(l[i]);
  };
  // a run's slots along the chain (none after a missing link) and hops
  struct Run {
    uint32_t slot[kRun];
    GHop hop[kRun][kParts];
  };
  SlotMap maps[kRun];
  auto load_run = [&](uint32_t c, uint32_t slot, Run* r) {
    if (per > kRun) load_maps(c, maps);  // else they are still there
#pragma unroll
    for (uint32_t i = 0; i < kRun; ++i) {
      r->slot[i] = slot;
      slot = map_bytes(maps[i], slot) & 255u;
    }
#pragma unroll
    for (uint32_t i = 0; i < kRun; ++i) {
      const uint32_t s = r->slot[i] < kSlots ? r->slot[i] : 0u;
      const GHop* h = pl.hops + (static_cast<uint64_t>(sp.chunk0 + (c + i < c1 ? c + i : c)) * kSlots + s) * kParts;
#pragma unroll
      for (uint32_t j = 0; j < kParts; ++j) r->hop[i][j] = h[j];
    }
    return slot;
  };
  uint32_t s[4], slot0, exit_slot;  // the slots by which the chain enters chunk c0 and the last one
  Run run;
  for (;;) {  // once, and again after each break that is mended
    run = Run{};  // no registers for these across a mend
    for (uint32_t i = 0; i < kRun; ++i) maps[i] = kSameSlots;
    SlotMap mine = kSameSlots;
    for (uint32_t c = c0; c < c1; c += kRun) {
      load_maps(c, maps);
#pragma unroll
      for (uint32_t i = 0; i < kRun; ++i)
        if (c + i < c1) mine = map_then(mine, maps[i]);
    }
    const uint32_t m[2] = {mine.lo, mine.hi}, same[2] = {kSameSlots.lo, kSameSlots.hi};
    uint32_t below[2], all_map[2];
    scan<LANES, 2>(m, same, [](uint32_t (&x)[2], const uint32_t (&y)[2]) {
      const SlotMap r = map_then(SlotMap{x[0], x[1]}, SlotMap{y[0], y[1]});
      x[0] = r.lo;
      x[1] = r.hi;
    }, lds, below, all_map);
    slot0 = below[0] & 255u;
    exit_slot = all_map[0] & 255u;
    for (int d = 0; d < 4; ++d) s[d] = 0;
    uint32_t slot = slot0, broken = 0xFFFFFFFFu, broken_slot = 0;  // the first chunk whose link is missing
    for (uint32_t c = c0; c < c1 && broken == 0xFFFFFFFFu; c += kRun) {
      const uint32_t next = load_run(c, slot, &run);
#pragma unroll
      for (uint32_t i = 0; i < kRun; ++i) {
        if (c + i >= c1 || run.slot[i] >= kSlots) continue;
#pragma unroll
        for (uint32_t j = 0; j < kParts; ++j) {
          s[0] += run.hop[i][j].blocks;
          for (int d = 0; d < 3; ++d) s[1 + d] += run.hop[i][j].dc[d];
        }
        const uint32_t after = i + 1 < kRun ? run.slot[i + 1] : next;
        if (after >= kSlots) {
          broken = c + i;
          broken_slot = run.slot[i];
        }
      }
      slot = next;
    }
    if (exit_slot < kSlots) break;  // the same for the whole group
    // every slot past the first break is none, so one lane has found one
    if (broken != 0xFFFFFFFFu) {
      atomicAdd(&pl.counters[kMended], 1u);
      mend_chain(pl, sp, jb, bytes, last, broken, broken_slot);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    if constexpr (LANES > 64) __syncthreads();
    else __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  }
  uint32_t at[4], all[4];
  const uint32_t zero[4] = {0, 0, 0, 0};
  scan<LANES, 4>(s, zero, [](uint32_t (&x)[4], const uint32_t (&y)[4]) {
    for (int i = 0; i < 4; ++i) x[i] += y[i];
  }, lds, at, all);
  // `state`: where part `part` of chunk c begins; n: its blocks
  auto task = [&](uint32_t c, uint32_t part, uint32_t state, uint32_t n, const uint32_t before[4]) {
    const uint32_t done = before[0] < iv.n_blocks ? before[0] : iv.n_blocks;
    GTask k;
    k.iv = sp.iv;
    k.word = c * kChunkWords + part * (kPart / 4) + (state >> 8);
    k.bit_b = ((state >> 3) & 31u) | (state & 7u) << 8;
    k.block0 = iv.block0 + done;
    k.n_blocks = n < iv.n_blocks - done ? n : iv.n_blocks - done;
    for (int d = 0; d < 3; ++d) {
      k.dc[d] = static_cast<uint16_t>(before[1 + d]);
      k.pad[d] = 0;
    }
    pl.tasks[static_cast<uint64_t>(sp.chunk0 + c) * kParts + part] = k;
  };
  auto entry = [&](uint32_t c, uint32_t in) {
    return in < kSlots ? pl.states[static_cast<uint64_t>(sp.chunk0 + c) * kSlots + in] & ~kGuessed : 0u;
  };
  uint32_t slot = slot0;
  for (uint32_t c = c0; c < c1; c += kRun) {
    if (per > kRun) slot = load_run(c, slot, &run);  // else it is still there
    uint32_t state[kRun];
#pragma unroll
    for (uint32_t i = 0; i < kRun; ++i) state[i] = entry(c + i < c1 ? c + i : c, run.slot[i]);
#pragma unroll
    for (uint32_t i = 0; i < kRun; ++i) {
      if (c + i >= c1) continue;
      uint32_t st = state[i];
#pragma unroll
      for (uint32_t j = 0; j < kParts; ++j) {
        task(c + i, j, st, run.hop[i][j].blocks, at);
        st = run.hop[i][j].state;
        at[0] += run.hop[i][j].blocks;
        for (int d = 0; d < 3; ++d) at[1 + d] += run.hop[i][j].dc[d];
      }
    }
  }
  // the last chunk's first part decodes all blocks that are left
  for (uint32_t c = last + id; c < sp.n_chunks; c += LANES)
    for (uint32_t j = 0; j < kParts; ++j) {
      if (c == last && j == 0) task(c, 0, entry(c, exit_slot), iv.n_blocks, all);
      else task(c, j, 0, 0, all);
    }
}

// ---- decoding ------------------------------------------------------------------------
// One lane decodes one interval, or one part of a split one, one symbol per
// step.  A block is built in 128 bytes of LDS (the value of a step is stored
// in the next one, beside its table lookup, so that only that lookup's
// latency is on the lane's chain); a lane whose block is complete waits for
// the next of the points that come every four steps, where it adds the DC
// prediction and the wave stores all complete blocks together, eight lanes a
// block, in whole 128-byte lines that do not stay in the L2.  When every lane
// stored its own blocks as they ended, three lanes of a wave did so in each
// step and all 64 waited for their 24 memory instructions.
// Bound by a lane's chain of steps where intervals are few, by issue and LDS
// (three workgroups a CU) where they are many: 153,904 intervals of 267 MB
// take 1.6 ms (3.4 with stuffed bytes and stores by lane), 1.3 million of 274
// MB 1.7 ms (2.5).

// Per-lane block buffers sit 128 bytes apart; their 16-byte parts are rotated
// by the lane, which spreads the lanes' stores over the banks.
struct BlockBuf {
  uint32_t base, rot;  // byte offset of the lane's buffer, 16 * (lane & 7)
  __device__ uint32_t at(uint32_t byte) const { return base | ((byte + rot) & 127u); }
};

constexpr int kDecodeSteps = 4;  // between two points; every second one refills

template <bool SPLIT>
__global__ __launch_bounds__(kThreads, 3) void entropy_decode(const GPlan pl) {
  __shared__ __align__(16) FastTables tables;
  __shared__ __align__(16) uint8_t block_bytes[kThreads * 128];
  __shared__ uint32_t words_mem[kRingWords * kThreads];
  __shared__ uint32_t list_mem[kThreads];  // block | lane << 28 (its low four bits) of the wave's complete blocks
  __shared__ int s_next;
  const uint32_t tid = threadIdx.x, lane = lane_of();
  const uint32_t wave = uniform(tid >> 6), wave0 = wave * 64;
  lds_tables* tabs = (lds_tables*)&tables;
  lds8* blocks = (lds8*)block_bytes;
  lds32* list = (lds32*)list_mem + wave0;
  const lds8* nat2 = (const lds8*)tables.nat2;  // indexed by the position after the coefficient
  const BlockBuf buf{tid * 128, (lane & 7u) * 16};
#pragma unroll
  for (uint32_t i = 0; i < 8; ++i) *reinterpret_cast<lds128*>(blocks + buf.base + 16 * i) = v4i_t{0, 0, 0, 0};
  uint32_t cur_job = 0xFFFFFFFFu;
  const uint32_t n_items = SPLIT ? pl.n_split_items : pl.pass.n_items;
  const GItem* items = pl.items + (SPLIT ? 0 : pl.n_split_items + pl.pass.item0);
  unsigned* counters = pl.counters + (SPLIT ? 0 : 2);
  for (;;) {
    if (tid == 0) s_next = static_cast<int>(atomicAdd(&counters[0], 1u));
    __syncthreads();
    const uint32_t it = uniform(static_cast<uint32_t>(s_next));
    __syncthreads();  // every lane has read s_next (and finished the last item)
    if (it >= n_items) break;
    const GItem item = items[it];
    const uint32_t job = uniform(item.job);
    const GJob& jb = pl.jobs[job];
    if (job != cur_job) {
      load_tables<kThreads>(jb.tables, tabs);
      __syncthreads();
      cur_job = job;
    }
    const uint32_t bpm = jb.bpm, comp_bits = jb.comp_bits, slots_dc = jb.dc_slots, slots_ac = jb.ac_slots;
    const GCodes* codes = jb.codes;
    gout128* coef = (gout128*)jb.coef;
    // the lane's task
    uint32_t which = 0, b = 0, block = 0, left = 0, block0 = 0, bytes = 0;
    uint32_t p0 = 0, p1 = 0, p2 = 0;
    const bool have_task = tid < item.count;
    WordRing words;
    words.base = (lds32*)words_mem + tid;
    words.src = (gin128*)pl.data;
    words.loading = false;
    words.have = words.last = 0;
    BitWindow w{0, 0, 0, 0};
    if (have_task) {
      uint32_t word = 0, bit = 0;
      which = item.first + tid;
      if constexpr (SPLIT) {
        const GTask k = pl.tasks[which];
        which = k.iv;
        word = k.word;
        bit = k.bit_b & 255u;
        b = k.bit_b >> 8;
        block = k.block0;
        left = k.n_blocks;
        p0 = k.dc[0];
        p1 = k.dc[1];
        p2 = k.dc[2];
      }
      const GInterval iv = pl.ivs[which];
      bytes = pl.bytes[which];
      block0 = iv.block0;
      if constexpr (!SPLIT) {
        block = block0;
        left = iv.n_blocks;
      }
      words.src = (gin128*)(pl.data + static_cast<uint64_t>(iv.dst) * 16);
      w = words.open(bytes, word, bit);
    }
    // k is the position of the block's next coefficient, at least 64 once it
    // is complete, kIdle in a lane that has nothing to do
    constexpr uint32_t kIdle = 1u << 20;
    uint32_t k = left > 0 ? 0u : kIdle, size = 0;
    uint32_t t = table_of(slots_dc, b), ac = table_of(slots_ac, b);
    uint32_t place = 126;  // where the last symbol's value goes: not yet stored
    int32_t value = 0, dc_value = 0;
    bool refill = true;
    const auto step = [&](uint32_t next) {
      const uint32_t top = w.top();
      uint32_t e = fast_entry(tabs, t, top);
      *reinterpret_cast<ldsi16*>(blocks + buf.at(place)) = static_cast<int16_t>(value);
      if ((e & 31u) == 0) e = long_code(tabs, codes, t, top, e, k != 0);
      size = e >> 5 & 15u;
      value = entry_value(top, e & 31u, size);
      dc_value = k == 0 ? value : dc_value;
      k += e >> 9;
      place = nat2[k];
      t = ac;
      w.drop(e & 31u, next);
    };
    while (__ballot(k < kIdle)) {
      if (refill) words.refill(k < kIdle, w.wi);
      refill = !refill;
#pragma unroll
      for (int s = 0; s < kDecodeSteps; ++s)
        if (k < 64 && words.ready(w.wi)) step(words.word(w.wi));
      const bool full = k >= 64 && k < kIdle;
      const uint64_t m = __ballot(full);
      if (m == 0) continue;
      if (full) {
        *reinterpret_cast<ldsi16*>(blocks + buf.at(place)) = static_cast<int16_t>(value);
        const uint32_t comp = comp_bits >> (2 * b) & 3u;
        const uint32_t p = (comp == 0 ? p0 : comp == 1 ? p1 : p2) + static_cast<uint32_t>(dc_value);
        *reinterpret_cast<ldsi16*>(blocks + buf.at(0)) = static_cast<int16_t>(p);
        p0 = comp == 0 ? p : p0;
        p1 = comp == 1 ? p : p1;
        p2 = comp == 2 ? p : p2;
        list[lanes_below(m)] = block | lane << 28;
        // a size with a position past the block's end: no code began, or a
        // run left the block
        uint32_t error = k > 64 && size ? (k >= kBadStep ? kBadCode : kBadRun) : kOk;
        b = b + 1 < bpm ? b + 1 : 0;
        if (b == 0 && error == kOk && static_cast<int64_t>(w.wi - 1u) * 32 - w.sh > static_cast<int64_t>(bytes) * 8)
          error = kOverrun;
        if (error) atomicMin(&pl.status[which], (block - block0) << 2 | error);
        ++block;
        --left;
        k = left > 0 && error == kOk ? 0u : kIdle;
        t = table_of(slots_dc, b);
        ac = table_of(slots_ac, b);
        place = 126;
        value = 0;
      }
      wave_sync();
      // the lanes are listed in order: how many lie in each 16 gives the
      // other two bits of a listed lane
      const uint32_t n = static_cast<uint32_t>(__builtin_popcountll(m));
      const uint32_t n1 = static_cast<uint32_t>(__builtin_popcountll(m & 0xFFFFull)),
                     n2 = static_cast<uint32_t>(__builtin_popcountll(m & 0xFFFFFFFFull)),
                     n3 = static_cast<uint32_t>(__builtin_popcountll(m & 0xFFFFFFFFFFFFull));
      for (uint32_t i = lane >> 3; i < n; i += 8) {
        const uint32_t x = list[i];
        const uint32_t from = x >> 28 | (i >= n2 ? 32u + (i >= n3 ? 16u : 0u) : i >= n1 ? 16u : 0u), part = lane & 7u;
        lds128* src = reinterpret_cast<lds128*>(blocks + ((wave0 + from) * 128 | ((16 * part + 16 * (from & 7u)) & 127u)));
        __builtin_nontemporal_store(*src, &coef[static_cast<uint64_t>(x & 0xFFFFFFFu) * 8 + part]);
        *src = v4i_t{0, 0, 0, 0};
      }
      wave_sync();
    }
  }
  // The last workgroup out rearms the queue for the next launch.  No fence:
  // each workgroup's own requests have returned before it reports, and a fence
  // here writes back the whole L2 of its XCD, once a workgroup, while others
  // still store.
  if (tid == 0) {
    const unsigned done = atomicAdd(&counters[1], 1u);
    if (done == gridDim.x - 1) {
      atomicExch(&counters[0], 0u);
      atomicExch(&counters[1], 0u);
    }
  }
}

}  // namespace gent
}  // namespace mjd

struct mjd_entropy_batch {
  mjd_ctx* ctx = nullptr;
  mjd::gent::GPlan plan{};
  std::vector<mjd::gent::GPass> passes;
  int grid = 0, split_grid = 0;          // workgroups of a decoding launch, at most
  uint8_t* d_mem = nullptr;              // every table and buffer of the plan
  std::vector<uint32_t> first_interval;  // per job, into the interval list
  std::vector<uint32_t> iv_index;        // per listed interval, its number in its scan
  uint64_t bytes = 0, chunks = 0;
};

namespace mjd {
namespace gent {

// The parts of one device allocation, in order; offsets are multiples of 256.
struct Layout {
  uint64_t size = 0;
  uint64_t add(uint64_t bytes) {
    const uint64_t at = size;
    size = (size + bytes + 255) & ~uint64_t{255};
    return at;
  }
};

// Bytes on the host that are not cleared, and that grow without a copy where
// they are many.
class HostBytes {
 public:
  HostBytes() = default;
  HostBytes(const HostBytes&) = delete;
  ~HostBytes() { free(bytes_); }
  void resize(size_t n) {
    uint8_t* p = static_cast<uint8_t*>(realloc(bytes_, n));
    if (!p) throw std::bad_alloc();
    bytes_ = p;
  }
  uint8_t* at(uint64_t offset) { return bytes_ + offset; }

 private:
  uint8_t* bytes_ = nullptr;
};

// The length above which intervals are split: the power of two (or none)
// that gives the batch the least time by these rates, all measured on 4:2:0
// files of quality 85 (us, with B and MB the entropy-coded bytes):
// - a lane that decodes a whole interval takes 0.41 us a byte, however few
//   there are (188 intervals of 14 KB: 7780 us, 9619 of 1.8 KB: 1000 us), and
//   a batch of them at least 5.5 us a MB (1.3 million intervals of 0.2 KB:
//   1740 us for 274 MB);
// - a split batch takes 110 us more than 12.5 us a MB (2.5 MB: 165 us, 36 MB:
//   531, where whole intervals of 1.9 KB take 957; 77 MB: 1067 against 1026;
//   211 MB: 2740).
// Splitting is for what fits kSplitMost, which bounds its memory: a split byte
// takes one of data and 2.8 of tables, and a job's skip tables count as the
// bytes that take as much.
constexpr uint64_t kSplitMost = uint64_t{256} << 20;
constexpr uint64_t kSkipBytes = kTableSlots * kSkipEntries * sizeof(uint16_t);
static uint32_t split_threshold(const std::vector<GInterval>& ivs, uint32_t* longest_of_all) {
  uint64_t bytes[33] = {};  // of the intervals of 2^(i-1) < length <= 2^i
  uint64_t count[33] = {};
  uint64_t jobs[33] = {};  // whose longest interval is one of them
  uint32_t longest[33] = {};
  for (size_t k = 0; k < ivs.size(); ++k) {
    const uint32_t len = ivs[k].end - ivs[k].start;
    const int i = len > 1 ? 32 - __builtin_clz(len - 1) : 0;
    bytes[i] += len;
    ++count[i];
    if (k == 0 || ivs[k - 1].job != ivs[k].job) ++jobs[i];  // a job's longest comes first
    longest[i] = std::max(longest[i], len);
  }
  *longest_of_all = *std::max_element(longest, longest + 33);
  double best = 0;
  uint32_t over = 0xFFFFFFFFu;
  uint64_t split = 0, skips = 0, rest = 0;
  for (int i = 0; i <= 32; ++i) rest += bytes[i];
  for (int i = 32; i >= 7; --i) {  // all above 2^i are split
    uint32_t most = 0;
    for (int j = 0; j <= i; ++j) most = std::max(most, longest[j]);
    const double t = (split ? 110.0 + 12.5e-6 * static_cast<double>(split) : 0.0) +
                     std::max(0.41 * most, 5.5e-6 * static_cast<double>(rest));
    if (split + skips <= kSplitMost && (i == 32 || t < best)) {
      best = t;
      over = i == 32 ? 0xFFFFFFFFu : 1u << i;
    }
    split += bytes[i] + count[i] * 2 * kChunk;
    skips += jobs[i] * (kSkipBytes / 4);
    rest -= bytes[i];
  }
  return over;
}

// How a batch is decoded, from its list of intervals: each job's one after the
// other, longest first.
struct Schedule {
  std::vector<GTile> tiles;
  std::vector<GSplit> splits;
  std::vector<GGroup> groups, more_groups;
  std::vector<GItem> items, split_items;
  std::vector<uint32_t> skip_jobs, split_of;
  std::vector<GPass> passes;
  uint64_t chunks = 0;  // of split intervals
  uint64_t units = 0;   // of 16 bytes of data
  uint32_t n_long = 0;
  bool many = false;
};

// The passes' data takes kPassBytes at most, or one interval's.  A pass ends
// with a round of workgroups that does not fill the chip, which a corpus of
// small files notices: 4096 of 80 KB with a marker per MCU row take 13.3 ms in
// one pass, 15.7 in two of 256 MiB.
constexpr uint64_t kPassBytes = uint64_t{1} << 30;
// lanes of the largest entropy_destuff: a wave per interval and tile, and the
// skip tables' (a launch's lanes are counted in 32 bits)
static_assert((kPassBytes / kPad + kSplitMost / (2 * kChunk) + (kPassBytes + kSplitMost) / kTile) * 64 +
                  kSplitMost / (kSkipBytes / 4) * (kSkipBytes / 2) < 0xFFFFFFFFu,
              "a launch holds a pass");

// Intervals above split_over are split, the others take passes of pass_bytes.
static void schedule(std::vector<GInterval>& ivs, const std::vector<uint32_t>& first_interval,
                     const std::vector<GJob>& gj, int cus, uint32_t split_over, uint64_t pass_bytes, Schedule* out) {
  Schedule& sc = *out;
  const size_t n = gj.size(), n_iv = ivs.size();
  // Split intervals lie in whole chunks, so that chunk i of the batch is at
  // byte i * kChunk of the data; the others follow them.
  for (size_t k = 0; k < n_iv && split_over != 0xFFFFFFFFu; ++k)
    if (ivs[k].end - ivs[k].start > split_over) sc.chunks += (static_cast<uint64_t>(ivs[k].end - ivs[k].start) + kPad) / kChunk + 1;
  const uint64_t base = sc.chunks ? (sc.chunks * kChunk + kTail) / 16 : 0;
  uint64_t units = base;
  uint32_t n_chunks = 0;
  sc.split_of.reserve(sc.chunks);
  sc.many = sc.chunks > uint64_t{FollowShape<false>::RESIDENT * FollowShape<false>::GROUP} * static_cast<uint64_t>(cus);
  GPass pass{};
  const auto close_pass = [&](size_t end) {
    pass.n_iv = static_cast<uint32_t>(end) - pass.iv0;
    pass.n_tiles = static_cast<uint32_t>(sc.tiles.size()) - pass.tile0;
    pass.n_items = static_cast<uint32_t>(sc.items.size()) - pass.item0;
    // longest items first, so that the last ones to start are short
    std::stable_sort(sc.items.begin() + pass.item0, sc.items.end(),
                     [](const GItem& x, const GItem& y) { return x.bytes > y.bytes; });
    sc.passes.push_back(pass);
    pass = GPass{static_cast<uint32_t>(end), 0, static_cast<uint32_t>(sc.tiles.size()), 0,
                 static_cast<uint32_t>(sc.items.size()), 0};
    sc.units = std::max(sc.units, units);
    units = base;
  };
  for (size_t j = 0; j < n; ++j) {
    const size_t end = j + 1 < n ? first_interval[j + 1] : n_iv;
    const uint32_t job = static_cast<uint32_t>(j), first_chunk = n_chunks;
    GItem item{job, 0, 0, 0};
    const auto close_item = [&] {
      if (item.count) sc.items.push_back(item);
      item.count = 0;
    };
    for (size_t k = first_interval[j]; k < end; ++k) {
      GInterval& iv = ivs[k];
      const uint32_t len = iv.end - iv.start;
      if (len > split_over) {
        const uint32_t c = static_cast<uint32_t>((static_cast<uint64_t>(len) + kPad) / kChunk + 1);
        iv.dst = n_chunks * (kChunk / 16);
        sc.split_of.insert(sc.split_of.end(), c, static_cast<uint32_t>(sc.splits.size()));
        sc.splits.push_back(GSplit{static_cast<uint32_t>(k), n_chunks, c});
        n_chunks += c;
      } else {
        const uint64_t u = (static_cast<uint64_t>(len) + kPad + 15) / 16;
        if (units > base && (units - base + u) * 16 > pass_bytes) {
          close_item();
          close_pass(k);
        }
        iv.dst = static_cast<uint32_t>(units);
        units += u;
        if (item.count == 0) {
          item.first = static_cast<uint32_t>(k);
          item.bytes = len;
        }
        if (++item.count == kThreads) close_item();
      }
      if (len > kTile) {
        const uint32_t first = static_cast<uint32_t>(sc.tiles.size()) - pass.tile0;
        for (uint32_t t = 0; t <= (len - 1) / kTile; ++t) sc.tiles.push_back(GTile{static_cast<uint32_t>(k), t, first});
      }
    }
    close_item();
    if (n_chunks > first_chunk) {
      sc.skip_jobs.push_back(job);
      const uint32_t parts = n_chunks * kParts;
      uint32_t per = std::min(kGuessThreads / gj[j].bpm, kGuessGroup);
      for (uint32_t f = first_chunk; f < n_chunks; f += per) sc.groups.push_back(GGroup{job, f, std::min(per, n_chunks - f)});
      per = sc.many ? FollowShape<true>::GROUP : FollowShape<false>::GROUP;
      for (uint32_t f = first_chunk; f < n_chunks; f += per) sc.more_groups.push_back(GGroup{job, f, std::min(per, n_chunks - f)});
      for (uint32_t f = first_chunk * kParts; f < parts; f += kThreads)
        sc.split_items.push_back(GItem{job, f, std::min<uint32_t>(kThreads, parts - f), kPart});
    }
  }
  close_pass(n_iv);
  // a workgroup of its own resolves each long split interval, so these come first
  std::vector<uint32_t> order(sc.splits.size()), place(sc.splits.size());
  for (size_t k = 0; k < order.size(); ++k) order[k] = static_cast<uint32_t>(k);
  const auto is_long = [&](uint32_t k) { return sc.splits[k].n_chunks > kLongSplit; };
  sc.n_long = static_cast<uint32_t>(std::stable_partition(order.begin(), order.end(), is_long) - order.begin());
  if (sc.n_long && sc.n_long < sc.splits.size()) {
    std::vector<GSplit> sorted(sc.splits.size());
    for (size_t k = 0; k < order.size(); ++k) {
      sorted[k] = sc.splits[order[k]];
      place[order[k]] = static_cast<uint32_t>(k);
    }
    sc.splits.swap(sorted);
    for (uint32_t& k : sc.split_of) k = place[k];
  }
}

static int build(mjd_ctx* ctx, const mjd_entropy_job* jobs, size_t n, mjd_entropy_batch* b) {
  if (n == 0) return fail(MJD_EINVAL, "empty entropy batch");
  if (n > (1u << 24)) return fail(MJD_EINVAL, "entropy batch of %zu jobs too large", n);
  std::vector<GJob> gj(n);
  // what is uploaded, the tables first: they are built where they go from
  Layout mem;
  const uint64_t o_tables = mem.add(n * sizeof(FastTables)), o_codes = mem.add(n * sizeof(GCodes[kTableSlots]));
  const Layout after_tables = mem;
  HostBytes host;
  host.resize(mem.size);
  std::vector<GInterval> ivs;
  uint64_t want = 0;  // as the scans say, which are not checked yet
  for (size_t j = 0; j < n; ++j) want += jobs[j].scan ? jobs[j].scan->n_intervals : 0;
  ivs.reserve(std::min<uint64_t>(want, 1u << 20));
  b->first_interval.resize(n);
  for (size_t j = 0; j < n; ++j) {
    const mjd_entropy_job& J = jobs[j];
    if (!J.scan || !J.h_offsets || !J.d_jpg || !J.d_coef)
      return fail(MJD_EINVAL, "job %zu: null scan, offsets, stream or coefficient pointer", j);
    if ((reinterpret_cast<uintptr_t>(J.d_jpg) & 15) || (reinterpret_cast<uintptr_t>(J.d_coef) & 15))
      return fail(MJD_EINVAL, "job %zu: stream or coefficients not 16-byte aligned", j);
    if (J.len > kMaxStream) return fail(MJD_EINVAL, "job %zu: stream of %llu bytes is too long", j,
                                        static_cast<unsigned long long>(J.len));
    host::ScanLayout L;
    int rc = host::scan_layout(J.scan, &L);
    if (rc != MJD_OK) {
      const std::string why = mjd_last_error();
      return fail(rc, "job %zu: %s", j, why.c_str());
    }
    if (L.bpm > static_cast<int>(kGuesses)) return fail(MJD_EINVAL, "job %zu: %d blocks per MCU", j, L.bpm);
    uint32_t tsel;
    FastTables* ft = reinterpret_cast<FastTables*>(host.at(o_tables)) + j;
    rc = tables_for(*J.scan, reinterpret_cast<GCodes*>(host.at(o_codes)) + kTableSlots * j, ft->t, &tsel);
    if (rc != MJD_OK) {
      const std::string why = mjd_last_error();
      return fail(rc, "job %zu: %s", j, why.c_str());
    }
    gj[j] = GJob{J.d_jpg, J.d_coef, nullptr, nullptr, nullptr, static_cast<uint32_t>(L.bpm), 0, 0, 0};
    build_places(host::zigzag_to_natural(), ft->nat2);
    for (int i = 0; i < L.bpm; ++i) {
      const uint32_t c = static_cast<uint32_t>(L.comp_of[i]);
      gj[j].comp_bits |= c << (2 * i);
      gj[j].dc_slots |= (tsel >> (4 * c) & 3u) << (2 * i);
      gj[j].ac_slots |= (tsel >> (4 * c + 2) & 3u) << (2 * i);
    }
    // the intervals: byte ranges from the restart index, checked against the stream
    const uint32_t ni = J.scan->n_intervals;
    const uint64_t ri = J.scan->restart_interval ? J.scan->restart_interval : L.n_mcus;
    const uint64_t* off = J.h_offsets;
    if (off[ni] > J.len) return fail(MJD_EINVAL, "job %zu: restart index past the stream end", j);
    const size_t first = ivs.size();
    b->first_interval[j] = static_cast<uint32_t>(first);
    if (first + ni > 0x7FFFFFF0u) return fail(MJD_EINVAL, "entropy batch holds too many intervals");
    for (uint32_t s = 0; s < ni; ++s) {
      if (off[s + 1] < off[s] + 2) return fail(MJD_EINVAL, "job %zu: restart index not increasing", j);
      GInterval iv;
      iv.start = static_cast<uint32_t>(off[s]);
      iv.end = static_cast<uint32_t>(off[s + 1] - 2);
      iv.dst = s;  // its number in the scan, until the list is sorted
      iv.block0 = static_cast<uint32_t>(s * ri * L.bpm);
      iv.n_blocks = static_cast<uint32_t>(std::min<uint64_t>(ri, L.n_mcus - s * ri) * L.bpm);
      iv.job = static_cast<uint32_t>(j);
      ivs.push_back(iv);
    }
    // A lane's decode time follows its interval's length, and a wave (and a
    // workgroup) lasts as long as its longest interval: sort the job's
    // intervals longest first so that each item holds intervals of similar
    // length.
    std::stable_sort(ivs.begin() + first, ivs.end(), [](const GInterval& x, const GInterval& y) {
      return x.end - x.start > y.end - y.start;
    });
    b->bytes += J.len;
  }
  const size_t n_iv = ivs.size();
  b->iv_index.resize(n_iv);
  for (size_t k = 0; k < n_iv; ++k) b->iv_index[k] = ivs[k].dst;
  int per_cu = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, entropy_decode<false>, kThreads, 0) != hipSuccess || per_cu < 1)
    per_cu = 1;
  const int cus = ctx->cu_count > 0 ? ctx->cu_count : 256;
  // One allocation: what the host fills first, then what the kernels write.
  // On a device with too little memory left for it the batch goes on without
  // splitting, then with smaller passes, down to one interval's data.
  uint32_t longest = 0;
  uint32_t split_over = split_threshold(ivs, &longest);
  uint64_t pass_bytes = kPassBytes;
  Schedule sc;
  uint64_t o_jobs, o_ivs, o_tiles, o_splits, o_groups, o_split_of, o_items, o_skip_jobs, o_counters,
      o_status, upload, o_bytes, o_kept, o_states, o_links, o_hops, o_tasks, o_skip, o_data;
  for (;;) {
    sc = Schedule{};
    schedule(ivs, b->first_interval, gj, cus, split_over, pass_bytes, &sc);
    mem = after_tables;
    o_jobs = mem.add(n * sizeof(GJob));
    o_ivs = mem.add(n_iv * sizeof(GInterval));
    o_tiles = mem.add(sc.tiles.size() * sizeof(GTile));
    o_splits = mem.add(sc.splits.size() * sizeof(GSplit));
    o_groups = mem.add((sc.groups.size() + sc.more_groups.size()) * sizeof(GGroup));
    o_split_of = mem.add(sc.split_of.size() * sizeof(uint32_t));
    o_items = mem.add((sc.split_items.size() + sc.items.size()) * sizeof(GItem));
    o_skip_jobs = mem.add(sc.skip_jobs.size() * sizeof(uint32_t));
    o_counters = mem.add(kCounters * sizeof(unsigned));
    o_status = mem.add(n_iv * sizeof(uint32_t));
    upload = mem.size;
    o_bytes = mem.add(n_iv * sizeof(uint32_t));
    o_kept = mem.add(sc.tiles.size() * sizeof(uint32_t));
    o_states = mem.add(sc.chunks * kSlots * sizeof(uint32_t));
    o_links = mem.add(sc.chunks * kSlots);
    o_hops = mem.add(sc.chunks * kSlots * kParts * sizeof(GHop));
    o_tasks = mem.add(sc.chunks * kParts * sizeof(GTask));
    o_skip = mem.add(sc.skip_jobs.size() * kSkipBytes);
    o_data = mem.add(sc.units * 16);
    if (hipMalloc(&b->d_mem, mem.size) == hipSuccess) break;
    b->d_mem = nullptr;
    (void)hipGetLastError();  // the launches ask for it
    if (split_over != 0xFFFFFFFFu) split_over = 0xFFFFFFFFu;
    else if (pass_bytes > std::max<uint64_t>(longest, 1u << 16)) pass_bytes /= 4;
    else return fail(MJD_ENOMEM, "device allocation for the entropy batch failed");
  }
  b->passes = sc.passes;
  b->chunks = sc.chunks;
  uint32_t most_items = 0;
  for (const GPass& ps : sc.passes) most_items = std::max(most_items, ps.n_items);
  b->grid = std::min<int>(static_cast<int>(most_items), per_cu * cus);
  b->split_grid = std::min<int>(static_cast<int>(sc.split_items.size()), per_cu * cus);
  uint8_t* d = b->d_mem;
  for (size_t j = 0; j < n; ++j) {
    gj[j].tables = reinterpret_cast<const FastTables*>(d + o_tables) + j;
    gj[j].codes = reinterpret_cast<const GCodes*>(d + o_codes) + kTableSlots * j;
  }
  for (size_t i = 0; i < sc.skip_jobs.size(); ++i)
    gj[sc.skip_jobs[i]].skip = reinterpret_cast<uint16_t*>(d + o_skip + i * kSkipBytes);
  host.resize(upload);
  auto fill = [&](uint64_t at, const auto& from) {
    const size_t bytes = from.size() * sizeof(from[0]);
    if (bytes) memcpy(host.at(at), from.data(), bytes);
    return at + bytes;
  };
  fill(o_jobs, gj);
  fill(o_ivs, ivs);
  fill(o_tiles, sc.tiles);
  fill(o_splits, sc.splits);
  fill(fill(o_groups, sc.groups), sc.more_groups);
  fill(o_split_of, sc.split_of);
  fill(fill(o_items, sc.split_items), sc.items);
  fill(o_skip_jobs, sc.skip_jobs);
  memset(host.at(o_counters), 0, kCounters * sizeof(unsigned));
  memset(host.at(o_status), 0xFF, n_iv * sizeof(uint32_t));  // kStatusOk
  if (hipMemcpy(d, host.at(0), upload, hipMemcpyHostToDevice) != hipSuccess)
    return fail(MJD_EDEVICE, "uploading the entropy batch tables failed");
  GPlan& p = b->plan;
  p.jobs = reinterpret_cast<const GJob*>(d + o_jobs);
  p.ivs = reinterpret_cast<const GInterval*>(d + o_ivs);
  p.tiles = reinterpret_cast<const GTile*>(d + o_tiles);
  p.splits = reinterpret_cast<const GSplit*>(d + o_splits);
  p.groups = reinterpret_cast<const GGroup*>(d + o_groups);
  p.split_of = reinterpret_cast<const uint32_t*>(d + o_split_of);
  p.items = reinterpret_cast<const GItem*>(d + o_items);
  p.skip_jobs = reinterpret_cast<const uint32_t*>(d + o_skip_jobs);
  p.n_skip = static_cast<uint32_t>(sc.skip_jobs.size());
  p.many = sc.many ? 1u : 0u;
  p.n_iv = static_cast<uint32_t>(n_iv);
  p.n_tiles = static_cast<uint32_t>(sc.tiles.size());
  p.n_groups = static_cast<uint32_t>(sc.groups.size());
  p.n_more_groups = static_cast<uint32_t>(sc.more_groups.size());
  p.n_splits = static_cast<uint32_t>(sc.splits.size());
  p.n_long = sc.n_long;
  p.n_items = static_cast<uint32_t>(sc.split_items.size() + sc.items.size());
  p.n_split_items = static_cast<uint32_t>(sc.split_items.size());
  p.data = d + o_data;
  p.bytes = reinterpret_cast<uint32_t*>(d + o_bytes);
  p.kept = reinterpret_cast<uint32_t*>(d + o_kept);
  p.status = reinterpret_cast<uint32_t*>(d + o_status);
  p.states = reinterpret_cast<uint32_t*>(d + o_states);
  p.links = d + o_links;
  p.hops = reinterpret_cast<GHop*>(d + o_hops);
  p.tasks = reinterpret_cast<GTask*>(d + o_tasks);
  p.counters = reinterpret_cast<unsigned*>(d + o_counters);
  return MJD_OK;
}

static void enqueue_splits(const GPlan& p, int grid, hipStream_t s) {
  const dim3 block(kThreads);
  hipLaunchKernelGGL(entropy_guess, dim3(p.n_groups), dim3(kGuessThreads), 0, s, p);
  if (p.many) hipLaunchKernelGGL(entropy_follow<true>, dim3(p.n_more_groups), dim3(FollowShape<true>::THREADS), 0, s, p);
  else hipLaunchKernelGGL(entropy_follow<false>, dim3(p.n_more_groups), dim3(FollowShape<false>::THREADS), 0, s, p);
  if (p.n_long) hipLaunchKernelGGL(entropy_resolve<1024>, dim3(p.n_long), dim3(1024), 0, s, p);
  const uint32_t rest = p.n_splits - p.n_long;
  if (rest) hipLaunchKernelGGL(entropy_resolve<64>, dim3((rest + kWaves - 1) / kWaves), block, 0, s, p);
  hipLaunchKernelGGL(entropy_decode<true>, dim3(grid), block, 0, s, p);
}

static hipError_t enqueue(const mjd_entropy_batch* b, hipStream_t s) {
  GPlan p = b->plan;
  const dim3 block(kThreads);
  for (size_t i = 0; i < b->passes.size(); ++i) {
    const GPass& ps = p.pass = b->passes[i];
    const bool last = i + 1 == b->passes.size();
    if (ps.n_tiles) hipLaunchKernelGGL(entropy_destuff_count, dim3((ps.n_tiles + kWaves - 1) / kWaves), block, 0, s, p);
    const uint32_t skip_groups = last ? p.n_skip * (kTableSlots * kSkipEntries / kThreads) : 0;
    hipLaunchKernelGGL(entropy_destuff, dim3((ps.n_iv + ps.n_tiles + kWaves - 1) / kWaves + skip_groups), block, 0, s, p);
    if (last && p.n_splits) enqueue_splits(p, b->split_grid, s);
    const uint32_t grid = std::min(static_cast<uint32_t>(b->grid), ps.n_items);
    if (grid) hipLaunchKernelGGL(entropy_decode<false>, dim3(grid), block, 0, s, p);
  }
  return hipGetLastError();
}

}  // namespace gent
}  // namespace mjd

extern "C" {

int mjd_entropy_batch_create(mjd_ctx* ctx, const mjd_entropy_job* jobs, size_t n, mjd_entropy_batch** out) {
  if (!ctx || !out) return mjd::fail(MJD_EINVAL, "null context or out-pointer");
  *out = nullptr;
  if (!jobs && n) return mjd::fail(MJD_EINVAL, "null jobs");
  int cur = 0;
  (void)hipGetDevice(&cur);
  if (cur != ctx->device && hipSetDevice(ctx->device) != hipSuccess)
    return mjd::fail(MJD_EDEVICE, "hipSetDevice(%d) failed", ctx->device);
  mjd_entropy_batch* b = new (std::nothrow) mjd_entropy_batch;
  if (!b) return mjd::fail(MJD_ENOMEM, "entropy batch allocation failed");
  b->ctx = ctx;
  int rc;
  try {
    rc = mjd::gent::build(ctx, jobs, n, b);
  } catch (const std::bad_alloc&) {
    rc = mjd::fail(MJD_ENOMEM, "host allocation for the entropy batch failed");
  }
  if (cur != ctx->device) (void)hipSetDevice(cur);
  if (rc != MJD_OK) {
    if (b->d_mem) (void)hipFree(b->d_mem);
    delete b;
    return rc;
  }
  *out = b;
  return MJD_OK;
}

int mjd_entropy_batch_launch(mjd_entropy_batch* b, void* stream) {
  if (!b) return mjd::fail(MJD_EINVAL, "null entropy batch");
  int cur = 0;
  (void)hipGetDevice(&cur);
  if (cur != b->ctx->device && hipSetDevice(b->ctx->device) != hipSuccess)
    return mjd::fail(MJD_EDEVICE, "hipSetDevice(%d) failed", b->ctx->device);
  const hipError_t e = mjd::gent::enqueue(b, static_cast<hipStream_t>(stream));
  if (cur != b->ctx->device) (void)hipSetDevice(cur);
  if (e != hipSuccess) return mjd::fail(MJD_EDEVICE, "entropy kernel launch failed: %s", hipGetErrorString(e));
  return MJD_OK;
}

int mjd_entropy_batch_status(mjd_entropy_batch* b, int64_t* bad_job) {
  if (!b) return mjd::fail(MJD_EINVAL, "null entropy batch");
  if (bad_job) *bad_job = -1;
  int cur = 0;
  (void)hipGetDevice(&cur);
  if (cur != b->ctx->device && hipSetDevice(b->ctx->device) != hipSuccess)
    return mjd::fail(MJD_EDEVICE, "hipSetDevice(%d) failed", b->ctx->device);
  std::vector<uint32_t> st(b->plan.n_iv);
  hipError_t e = hipDeviceSynchronize();
  if (e == hipSuccess) e = hipMemcpy(st.data(), b->plan.status, st.size() * sizeof(uint32_t), hipMemcpyDeviceToHost);
  if (cur != b->ctx->device) (void)hipSetDevice(cur);
  if (e != hipSuccess) return mjd::fail(MJD_EDEVICE, "reading the entropy status failed: %s", hipGetErrorString(e));
  for (uint32_t i = 0; i < b->plan.n_iv; ++i) {
    if (st[i] == mjd::gent::kStatusOk) continue;
    const auto it = std::upper_bound(b->first_interval.begin(), b->first_interval.end(), i);
    const int64_t job = static_cast<int64_t>(it - b->first_interval.begin()) - 1;
    if (bad_job) *bad_job = job;
    static const char* what[] = {"", "an invalid Huffman code", "a coefficient run past the end of a block",
                                 "an interval that ends before its last MCU"};
    return mjd::fail(MJD_ECORRUPT, "job %lld, restart interval %u: %s", static_cast<long long>(job),
                     b->iv_index[i], what[st[i] & 3u]);
  }
  return MJD_OK;
}

int mjd_entropy_batch_info(const mjd_entropy_batch* b, uint32_t* intervals, uint32_t* workgroups, uint64_t* bytes) {
  if (!b) return mjd::fail(MJD_EINVAL, "null entropy batch");
  if (intervals) *intervals = b->plan.n_iv;
  if (workgroups) *workgroups = static_cast<uint32_t>(b->grid + b->split_grid);
  if (bytes) *bytes = b->bytes;
  return MJD_OK;
}

int mjd_entropy_batch_splits(mjd_entropy_batch* b, uint32_t* split_intervals, uint64_t* chunks, uint32_t* mended) {
  if (!b) return mjd::fail(MJD_EINVAL, "null entropy batch");
  if (split_intervals) *split_intervals = b->plan.n_splits;
  if (chunks) *chunks = b->chunks;
  if (!mended) return MJD_OK;
  int cur = 0;
  (void)hipGetDevice(&cur);
  if (cur != b->ctx->device && hipSetDevice(b->ctx->device) != hipSuccess)
    return mjd::fail(MJD_EDEVICE, "hipSetDevice(%d) failed", b->ctx->device);
  hipError_t e = hipDeviceSynchronize();
  if (e == hipSuccess)
    e = hipMemcpy(mended, b->plan.counters + mjd::gent::kMended, sizeof(uint32_t), hipMemcpyDeviceToHost);
  if (cur != b->ctx->device) (void)hipSetDevice(cur);
  if (e != hipSuccess) return mjd::fail(MJD_EDEVICE, "reading the entropy batch failed: %s", hipGetErrorString(e));
  return MJD_OK;
}

void mjd_entropy_batch_destroy(mjd_entropy_batch* b) {
  if (!b) return;
  int cur = 0;
  (void)hipGetDevice(&cur);
  if (cur != b->ctx->device) (void)hipSetDevice(b->ctx->device);
  (void)hipDeviceSynchronize();
  if (b->d_mem) (void)hipFree(b->d_mem);
  if (cur != b->ctx->device) (void)hipSetDevice(cur);
  delete b;
}

}  // extern "C"
