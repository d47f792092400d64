// Compares the GPU entropy kernels' look-up tables with the canonical code of
// T.81 Annex C, for every 16-bit front of a stream.  Usage:
// entropy_tables_host <in.jpg>; prints the number of fronts checked, exit
// status 3 on a difference.
#include <stdio.h>
#include <stdlib.h>

#include <memory>
#include <vector>

#include "entropy_walk.h"
#include "mjd.h"

using namespace mjd::gent;

// The entry of the code at the front of the 16 bits `w`, from the DHT
// segment's counts and symbols alone.
static uint32_t reference(const mjd_huffman& h, bool ac, uint32_t w) {
  uint32_t code = 0, k = 0;
  for (uint32_t l = 1; l <= 16; ++l, code <<= 1)
    for (int i = 0; i < h.bits[l - 1]; ++i, ++code, ++k)
      if (w >> (16 - l) == code) {
        const uint32_t e = table_entry(l, h.vals[k], ac);
        return e ? e : kBadEntry;
      }
  return kBadEntry;
}

int main(int argc, char** argv) {
  if (argc != 2) return 2;
  FILE* f = fopen(argv[1], "rb");
  if (!f) return 2;
  std::vector<uint8_t> jpg;
  for (int c; (c = fgetc(f)) != EOF;) jpg.push_back(static_cast<uint8_t>(c));
  fclose(f);
  auto scan = std::make_unique<mjd_scan>();
  uint16_t qt[4][64];
  if (mjd_parse(jpg.data(), jpg.size(), scan.get(), qt) != MJD_OK) return 2;
  unsigned long checked = 0;
  for (int id = 0; id < 8; ++id) {
    const bool ac = id >= 4;
    const mjd_huffman& h = ac ? scan->ac[id - 4] : scan->dc[id];
    if (!h.defined) continue;
    auto g = std::make_unique<GHuff>();
    auto t = std::make_unique<FastTable>();
    if (build_gtable(h, ac, g.get()) != kTableOk) return 2;
    build_fast_table(*g, ac, t.get());
    const PlainTab plain{g.get()};
    const auto entry = [&](uint32_t top) {
      const uint32_t e = t->fast[top >> (32 - kGLook)];
      return e & 31u ? e : more_entry(e, top, ac, [&](uint32_t i) {
        if (i >= kMore) exit(3);
        return static_cast<uint32_t>(t->more[i]);
      }, plain, 0);
    };
    for (uint32_t w = 0; w < 65536; ++w, ++checked)
      if (entry(w << 16 | 0x5A5Au) != reference(h, ac, w)) {
        fprintf(stderr, "table %d, bits %04x: entry %x, not %x\n", id, w, entry(w << 16), reference(h, ac, w));
        return 3;
      }
    // a step of several symbols: the same bits and positions one by one,
    // whatever bits follow those it looked at
    for (uint32_t i = 0; i < kSkipEntries; ++i, ++checked) {
      const uint32_t m = skip_entry(i, ac, entry);
      for (uint32_t rest : {0u, 0x1FFFFFu, 0x155555u}) {
        const uint64_t front = (static_cast<uint64_t>(i << (32 - kSkipLook) | rest) << 32) | 0xA5A5A5A5u;
        uint32_t bits = 0, step = 0;
        bool eob = false;
        while (bits < (m & 31u)) {
          const uint32_t e = reference(h, ac, static_cast<uint32_t>(front << bits >> 48));
          if (e == kBadEntry || eob) return 3;
          eob = ac && e >> 9 == kEobStep;
          step += eob ? 0 : e >> 9;
          bits += e & 31u;
          if (!ac && (m >> 12) != (e >> 5 & 15u)) return 3;
        }
        if (bits == 0 ? m != kEobStep << 5 : bits != (m & 31u) || step != (m >> 5 & 63u) || eob != ((m >> 5 & kEobStep) != 0)) {
          fprintf(stderr, "table %d, skip entry %x: %u bits, %u on, eob %d, entry %x\n", id, i, bits, step, eob, m);
          return 3;
        }
        // past position 63 the whole entry holds if, and only if, it ends the block there
        for (uint32_t k : {0u, 1u, 30u, 62u, 63u}) {
          const uint32_t to = k + (m >> 5 & 127u);
          if (to > 63 && skip_takes_one(m, to) != (bits == 0 || !eob || k + step > 63)) return 3;
        }
      }
    }
  }
  printf("%lu\n", checked);
  return 0;
}
