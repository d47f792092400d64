// Pieces of the GPU entropy decoder that work on destuffed data: the zero
// byte that follows each 0xFF of a scan is dropped beforehand, so a lane
// takes its bits from plain words and one refill is one word.  Written for
// one lane, through a table interface, so that a CPU caller can run them too.
#pragma once

#include "entropy_lane.h"

namespace mjd {
namespace gent {

// A window of two words (most significant bit first) over a word stream.
// sh is the number of unread bits of w1's word that the 32-bit view leaves
// out, 0..31; wi is the word that follows w1.
struct BitWindow {
  uint32_t w0, w1, wi;
  int32_t sh;

  // The next 32 bits.
  MJD_HD uint32_t top() const {
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_alignbit(w0, w1, static_cast<uint32_t>(sh));
#else
    return static_cast<uint32_t>((static_cast<uint64_t>(w0) << 32 | w1) >> sh);
#endif
  }
  // Drops n <= 31 bits; `next` is word wi.
  MJD_HD void drop(uint32_t n, uint32_t next) {
    sh -= static_cast<int32_t>(n);
    const bool over = sh < 0;
    sh &= 31;
    w0 = over ? w1 : w0;
    w1 = over ? next : w1;
    wi += over ? 1u : 0u;
  }
  // Position of the next unread bit, modulo 2^32 (callers compare positions
  // that lie close together).
  MJD_HD uint32_t pos() const { return 32u * (wi - 1u) - static_cast<uint32_t>(sh); }
};

// First word that a window at bit position 32 * word + bit needs, and the
// window itself from words q - 1 and q (q = word, or word + 1 where bit > 0).
MJD_HD inline uint32_t window_word(uint32_t word, uint32_t bit) { return word + (bit ? 1u : 0u); }
MJD_HD inline BitWindow window_at(uint32_t word, uint32_t bit, uint32_t before, uint32_t at) {
  const uint32_t q = window_word(word, bit);
  return BitWindow{before, at, q + 1u, static_cast<int32_t>(32u * (q - word) - bit)};
}

// A Huffman table as the kernels keep it in LDS: one look-up by the next
// kGLook bits, and one more where the code is longer.  An entry of `fast`
// whose low five bits (the bits used) are zero leads to `more`:
//   bits 5-7    further bits of the code to look at, n
//   bits 8-15   half the index of the 2^n entries of that prefix
// so a prefix takes as many entries as its longest code needs.  Entry 0 of
// `more` is 0 and stands for a prefix that found no entries left: the
// canonical code's limits then decide (long_entry).  Where no code begins,
// the entry is kBadEntry: a magnitude size and a step that no valid entry has
// together, so that a lane needs no test of its own for it.
constexpr uint32_t kMore = 320;
constexpr uint32_t kBadStep = 127;
constexpr uint32_t kBadEntry = 16u | 15u << 5 | kBadStep << 9;
constexpr uint32_t kBadPrefix = 1u << 8;  // n = 0 at entry 2, kBadEntry
struct FastTable {
  uint16_t fast[1 << kGLook];
  uint16_t more[kMore];
};
// Positions past 63 (an EOB, or data that leaves the block) write to
// coefficient 63.
constexpr uint32_t kPlaces = 64 + kBadStep + 1;
struct FastTables {
  FastTable t[kTableSlots];
  uint8_t nat2[kPlaces];  // byte offset in a block (twice the natural index) of zig-zag position k - 1
};
static_assert(sizeof(FastTables) % 16 == 0, "tables copy as 16-byte chunks");

struct PlainTab {
  const GHuff* tab;
  MJD_HD uint32_t fast(int t, int i) const { return tab[t].fast[i]; }
  MJD_HD int lim(int t, int l) const { return tab[t].lim[l]; }
  MJD_HD int valoff(int t, int l) const { return tab[t].valoff[l]; }
  MJD_HD int val(int t, int i) const { return tab[t].vals[i]; }
};

// The same of the canonical code alone.
struct CodeTab {
  const GCodes* tab;
  MJD_HD int lim(int t, int l) const { return tab[t].lim[l]; }
  MJD_HD int valoff(int t, int l) const { return tab[t].valoff[l]; }
  MJD_HD int val(int t, int i) const { return tab[t].vals[i]; }
};

// Code by code (256 at most): a batch of many small files spends its time here.
inline void build_fast_table(const GCodes& h, bool ac, FastTable* f) {
  memset(f->more, 0, sizeof(f->more));
  f->more[2] = kBadEntry;
  uint32_t filled = 0;  // canonical codes follow each other from 0 on
  for_codes(h, ac, 1, kGLook, [&](uint32_t code, int l, uint32_t e) {
    const uint32_t end = (code + 1) << (kGLook - l);
    for (; filled < end; ++filled) f->fast[filled] = static_cast<uint16_t>(e ? e : kBadPrefix);
  });
  for (; filled < 1u << kGLook; ++filled) f->fast[filled] = static_cast<uint16_t>(kBadPrefix);
  uint32_t prefix = 1u << kGLook, bits = 0, used = 3;  // bits past the prefix of its longest code
  const auto place = [&] {
    if (prefix == 1u << kGLook) return;
    const uint32_t at = (used + 1u) & ~1u;
    if (at + (1u << bits) > kMore) {
      f->fast[prefix] = 0;
      return;
    }
    for (uint32_t v = 0; v < 1u << bits; ++v) f->more[at + v] = static_cast<uint16_t>(kBadEntry);
    f->fast[prefix] = static_cast<uint16_t>(bits << 5 | at >> 1 << 8);
    used = at + (1u << bits);
  };
  for_codes(h, ac, kGLook + 1, 16, [&](uint32_t code, int l, uint32_t e) {
    if (e == 0) return;
    const uint32_t n = static_cast<uint32_t>(l - kGLook);
    if (code >> n != prefix) {
      place();
      prefix = code >> n;
    }
    bits = n;  // never shorter than the codes before
  });
  place();
  for_codes(h, ac, kGLook + 1, 16, [&](uint32_t code, int l, uint32_t e) {
    const uint32_t n = static_cast<uint32_t>(l - kGLook), to = f->fast[code >> n];
    if (e == 0 || to == 0) return;
    const uint32_t m = to >> 5 & 7u, at = (to >> 8) * 2 + ((code & ((1u << n) - 1u)) << (m - n));
    for (uint32_t v = 0; v < 1u << (m - n); ++v) f->more[at + v] = static_cast<uint16_t>(e);
  });
}

inline void build_places(const uint8_t* natural, uint8_t nat2[kPlaces]) {
  for (uint32_t k = 0; k < kPlaces; ++k) nat2[k] = static_cast<uint8_t>(2 * natural[k == 0 ? 0 : k < 64 ? k - 1 : 63]);
}

// The whole entry at the front of `top`, from its `fast` entry e, which uses
// no bits; more(i) reads entry i of `more`.
template <class More, class Tab>
MJD_HD inline uint32_t more_entry(uint32_t e, uint32_t top, bool ac, const More& more, const Tab& tab, int t) {
  const uint32_t n = e >> 5 & 7u;
  const uint32_t m = more((e >> 8) * 2 + (static_cast<uint32_t>(static_cast<uint64_t>(top << kGLook) << n >> 32)));
  if (m) return m;
  const uint32_t l = long_entry(tab, t, top, ac);
  return l ? l : kBadEntry;
}

// Several symbols at once, for lanes that only look for block boundaries:
// what the next kSkipLook bits determine.
//   bits 0-4     bits of all its symbols, 0 where there is not even one
//   bits 5-11    how far they move the zig-zag position, and kEobStep more
//                where the last one is EOB or there is none
//   bits 12-15   DC: the magnitude size of its one symbol
// So a position past 63 is the one test a lane needs for the end of a block,
// for a code that the look-up does not hold and for symbols that together
// leave the block (skip_takes_one: these two take one symbol instead).
constexpr uint32_t kSkipLook = 11;
constexpr uint32_t kSkipEntries = 1u << kSkipLook;

template <class Entry>
MJD_HD inline uint32_t skip_entry(uint32_t index, bool ac, const Entry& entry) {
  const uint32_t top = index << (32 - kSkipLook);
  uint32_t bits = 0, step = 0;
  for (;;) {
    const uint32_t e = entry(top << bits);
    const uint32_t size = e >> 5 & 15u;
    if (e == kBadEntry || bits + (e & 31u) - size > kSkipLook) break;  // no code among the known bits
    if (!ac) return (e & 31u) | 1u << 5 | size << 12;
    if (e >> 9 == kEobStep) return (bits + (e & 31u)) | (step | kEobStep) << 5;
    if (step + (e >> 9) > 63) break;
    bits += e & 31u;
    step += e >> 9;
    if (bits >= kSkipLook) break;
  }
  return bits ? bits | step << 5 : kEobStep << 5;
}

// Of an entry that takes the position to `to`, past 63.
MJD_HD inline bool skip_takes_one(uint32_t m, uint32_t to) { return (m & 31u) == 0 || to - (m >> 5 & kEobStep) > 63; }

// The value whose `size` magnitude bits end `total` bits into `top` (T.81
// F.2.2.1 EXTEND); 0 for size 0.
MJD_HD inline int32_t entry_value(uint32_t top, uint32_t total, uint32_t size) {
#if defined(__HIP_DEVICE_COMPILE__)
  const int32_t raw = static_cast<int32_t>(__builtin_amdgcn_ubfe(top, 32u - total, size));
#else
  const int32_t raw = size ? static_cast<int32_t>((top >> (32u - total)) & ((1u << size) - 1u)) : 0;
#endif
  const int32_t mask = static_cast<int32_t>((1u << size) - 1u);
  return raw > (mask >> 1) ? raw : raw - mask;
}

// A split interval is cut into chunks of destuffed bytes.  A state names a
// block boundary at or after a byte of it: the bits from there, and the block
// of the MCU that begins at the boundary.
constexpr uint32_t kNoState = 0xFFFFFFFFu;
MJD_HD inline uint32_t make_state(uint32_t bits, uint32_t b) { return bits << 3 | b; }

// Slots of a chunk: the distinct exits of the chunk before it for the first
// blocks that are tried there, marked, and the boundaries that none of them
// reached, in the slots that are left (six on average for 4:2:0, at least two).
constexpr uint32_t kGuesses = 6, kSlots = 8;
constexpr uint32_t kGuessed = 1u << 31;
constexpr uint32_t kNoLink = 15;

// Maps of a chunk's slots to the next chunk's, a byte a slot, anything above
// 12 for no slot: the links as they are stored, with 8 to 12 (which no link
// is) made so, because a byte permute takes one map through another.
struct SlotMap {
  uint32_t lo, hi;  // slots 0-3, 4-7
};
constexpr SlotMap kSameSlots{0x03020100u, 0x07060504u};
MJD_HD inline uint32_t no_slot_above_7(uint32_t x) {
  const uint32_t b = x & 0x08080808u;
  return x | b >> 1 | b >> 2 | b >> 3;
}
MJD_HD inline SlotMap map_of_links(uint64_t links) {
  return SlotMap{no_slot_above_7(static_cast<uint32_t>(links)), no_slot_above_7(static_cast<uint32_t>(links >> 32))};
}
// For each byte of `slots`, what `m` maps it to.
MJD_HD inline uint32_t map_bytes(SlotMap m, uint32_t slots) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_perm(m.hi, m.lo, slots);
#else
  uint32_t r = 0;
  for (uint32_t i = 0; i < 4; ++i) {
    const uint32_t s = slots >> (8 * i) & 0xFFu;
    r |= (s < 4 ? m.lo >> (8 * s) & 0xFFu : s < kSlots ? m.hi >> (8 * (s - 4)) & 0xFFu : 0xFFu) << (8 * i);
  }
  return r;
#endif
}
// First `a`, then `b`.
MJD_HD inline SlotMap map_then(SlotMap a, SlotMap b) { return SlotMap{map_bytes(b, a.lo), map_bytes(b, a.hi)}; }

}  // namespace gent
}  // namespace mjd
