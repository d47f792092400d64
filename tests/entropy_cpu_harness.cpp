// The GPU entropy decoder's own source, host plan and kernels, on the CPU
// under a sanitizer (hip_on_cpu.h).  Every table and buffer of the plan is
// moved to memory of exactly its size before the launch, as are the streams
// and the coefficients, so an access outside any of them is reported.
//   entropy_cpu_harness [seed=N] [cus=N] [same=N] [largest=BYTES] file...
// decodes the files as the jobs of one batch (each `same` times), compares
// with the host decoder, and prints what the batch was made of.  Exit status
// 0: every status and coefficient as on the host.
#include <sanitizer/asan_interface.h>

#include "hip_on_cpu.h"

#include "mjd.h"
#include "mjd_common.h"

struct mjd_ctx {
  int device = 0;
  int cu_count = 256;
};

static unsigned long global_words;  // words that a lane read past its workgroup's copy
#define __builtin_expect(c, v) ((c) ? true : (++global_words, false))
#include "entropy_under_test.h"
#undef __builtin_expect

using namespace mjd::gent;

namespace {

std::vector<uint8_t> read_file(const char* path) {
  std::vector<uint8_t> d;
  FILE* f = fopen(path, "rb");
  if (!f) exit(2);
  for (int c; (c = fgetc(f)) != EOF;) d.push_back(static_cast<uint8_t>(c));
  fclose(f);
  return d;
}

// n elements in memory of their own, with the bytes that `from` holds.
template <class T, class P>
void move_out(P*& field, uint64_t n, std::vector<void*>* owned) {
  const uint64_t bytes = n * sizeof(T);
  void* p = aligned_alloc(16, bytes ? (bytes + 15) / 16 * 16 : 16);
  // aligned_alloc takes whole multiples; give the tail back to the sanitizer
  memcpy(p, reinterpret_cast<const void*>(field), bytes);
  ASAN_POISON_MEMORY_REGION(static_cast<char*>(p) + bytes, (bytes ? (bytes + 15) / 16 * 16 : 16) - bytes);
  field = reinterpret_cast<P*>(p);
  owned->push_back(p);
}

struct Image {
  std::vector<uint8_t> file;
  mjd_scan scan;
  std::vector<uint64_t> off;
  uint64_t n_blocks;
  std::vector<int16_t> host;
  bool ok;
  uint8_t* jpg;
  int16_t* coef;
};

}  // namespace

int main(int argc, char** argv) {
  mjd_ctx ctx;
  unsigned same = 1;
  std::vector<Image> images;
  for (int i = 1; i < argc; ++i) {
    if (!strncmp(argv[i], "seed=", 5)) cpu::options.seed = static_cast<unsigned>(atoi(argv[i] + 5));
    else if (!strncmp(argv[i], "cus=", 4)) ctx.cu_count = atoi(argv[i] + 4);
    else if (!strncmp(argv[i], "same=", 5)) same = static_cast<unsigned>(atoi(argv[i] + 5));
    else if (!strncmp(argv[i], "largest=", 8)) cpu::options.largest = strtoull(argv[i] + 8, nullptr, 10);
    else images.push_back(Image{read_file(argv[i]), {}, {}, 0, {}, false, nullptr, nullptr});
  }
  std::vector<mjd_entropy_job> jobs;
  std::vector<Image*> of;
  bool any_bad = false;
  for (Image& im : images) {
    uint16_t qt[4][64];
    if (mjd_parse(im.file.data(), im.file.size(), &im.scan, qt) != MJD_OK) {
      fprintf(stderr, "parse: %s\n", mjd_last_error());
      return 2;
    }
    im.off.resize(im.scan.n_intervals + 1);
    if (mjd_restart_index(im.file.data(), im.file.size(), &im.scan, im.off.data()) != MJD_OK) {
      fprintf(stderr, "restart index: %s\n", mjd_last_error());
      return 2;
    }
    mjd::host::ScanLayout L;
    if (mjd::host::scan_layout(&im.scan, &L) != MJD_OK) return 2;
    im.n_blocks = L.n_mcus * static_cast<uint64_t>(L.bpm);
    im.host.assign(im.n_blocks * 64, 0);
    im.ok = mjd_entropy_decode(im.file.data(), im.file.size(), &im.scan, im.off.data(), im.host.data(), 0, L.mcus_y, 1) == MJD_OK;
    any_bad = any_bad || !im.ok;
    const size_t padded = (im.file.size() + 15) / 16 * 16;
    im.jpg = static_cast<uint8_t*>(aligned_alloc(16, padded));
    memset(im.jpg, 0xFF, padded);
    memcpy(im.jpg, im.file.data(), im.file.size());
  }
  for (unsigned k = 0; k < same; ++k)
    for (Image& im : images) {
      int16_t* coef = static_cast<int16_t*>(aligned_alloc(16, im.n_blocks * 128));
      memset(coef, 0x5A, im.n_blocks * 128);
      jobs.push_back(mjd_entropy_job{&im.scan, im.off.data(), im.jpg, im.file.size(), coef});
      of.push_back(&im);
    }
  mjd_entropy_batch* b = nullptr;
  if (mjd_entropy_batch_create(&ctx, jobs.data(), jobs.size(), &b) != MJD_OK) {
    printf("create: %s\n", mjd_last_error());
    return 1;
  }
  const unsigned long long memory = cpu::options.allocated;
  const GPlan& plan = b->plan;
  uint64_t chunks = 0, bytes = 0;
  for (uint32_t i = 0; i < plan.n_splits; ++i) chunks += plan.splits[i].n_chunks;
  if (chunks) bytes = chunks * kChunk + kTail;
  for (uint32_t i = 0; i < plan.n_iv; ++i) {
    const GInterval& iv = plan.ivs[i];
    bytes = std::max<uint64_t>(bytes, static_cast<uint64_t>(iv.dst) * 16 + (iv.end - iv.start + kPad + 15) / 16 * 16);
  }
  std::vector<void*> owned;
  GPlan p = plan;
  const uint64_t n = jobs.size();
  move_out<GJob>(p.jobs, n, &owned);
  for (uint64_t j = 0; j < n; ++j) {
    GJob& jb = const_cast<GJob*>(p.jobs)[j];
    move_out<FastTables>(jb.tables, 1, &owned);
    move_out<GCodes>(jb.codes, kTableSlots, &owned);
    if (jb.skip) move_out<uint16_t>(jb.skip, kTableSlots * kSkipEntries, &owned);
  }
  move_out<GInterval>(p.ivs, p.n_iv, &owned);
  move_out<GTile>(p.tiles, p.n_tiles, &owned);
  move_out<GSplit>(p.splits, p.n_splits, &owned);
  move_out<GGroup>(p.groups, p.n_groups + p.n_more_groups, &owned);
  move_out<uint32_t>(p.split_of, chunks, &owned);
  move_out<GItem>(p.items, p.n_items, &owned);
  move_out<uint32_t>(p.skip_jobs, p.n_skip, &owned);
  move_out<uint8_t>(p.data, bytes, &owned);
  move_out<uint32_t>(p.bytes, p.n_iv, &owned);
  move_out<uint32_t>(p.kept, p.n_tiles, &owned);
  move_out<uint32_t>(p.status, p.n_iv, &owned);
  move_out<uint32_t>(p.states, chunks * kSlots, &owned);
  move_out<uint8_t>(p.links, chunks * kSlots, &owned);
  move_out<GHop>(p.hops, chunks * kSlots * kParts, &owned);
  move_out<GTask>(p.tasks, chunks * kParts, &owned);
  move_out<unsigned>(p.counters, kCounters, &owned);
  b->plan = p;
  int rc = 0;
  // what entropy_resolve finds: chains with a break, and those of them whose
  // next chunk has a slot left
  unsigned long breaks = 0, out_of_hops = 0, mended = 0;
  bool counted = false;
  cpu::before_launch = [&](const char* kernel) {
    if (strncmp(kernel, "entropy_resolve", 15) || counted) return;
    counted = true;
    for (uint32_t i = 0; i < p.n_splits; ++i) {
      const GSplit& sp = p.splits[i];
      const uint32_t len = p.bytes[sp.iv], last = len ? (len - 1) / kChunk : 0;
      uint32_t slot = 0;
      for (uint32_t c = 0; c < last; ++c) {
        slot = p.links[static_cast<uint64_t>(sp.chunk0 + c) * kSlots + slot];
        if (slot < kSlots) continue;
        const uint32_t* to = p.states + static_cast<uint64_t>(sp.chunk0 + c + 1) * kSlots;
        ++breaks;
        if (std::find(to, to + kSlots, kNoState) != to + kSlots) ++out_of_hops;
        break;
      }
    }
  };
  for (int rep = 0; rep < 2; ++rep) {
    if (mjd_entropy_batch_launch(b, nullptr) != MJD_OK) {
      printf("launch: %s\n", mjd_last_error());
      return 1;
    }
    uint32_t n_mended = 0;
    uint64_t n_chunks = 0;
    if (mjd_entropy_batch_splits(b, nullptr, &n_chunks, &n_mended) != MJD_OK || n_chunks != chunks) rc = 3;
    mended = n_mended;
    int64_t bad = -1;
    const int st = mjd_entropy_batch_status(b, &bad);
    if ((st != MJD_OK) != any_bad || (st != MJD_OK && of[static_cast<size_t>(bad)]->ok)) {
      printf("status %d, job %lld\n", st, static_cast<long long>(bad));
      rc = 3;
    }
    for (size_t j = 0; j < jobs.size(); ++j) {
      if (of[j]->ok && memcmp(jobs[j].d_coef, of[j]->host.data(), of[j]->n_blocks * 128)) {
        size_t k = 0;
        while (jobs[j].d_coef[k] == of[j]->host[k]) ++k;
        printf("job %zu of launch %d: block %zu, coefficient %zu\n", j, rep, k / 64, k % 64);
        rc = 3;
      }
      memset(jobs[j].d_coef, 0x33, of[j]->n_blocks * 128);
    }
  }
  printf("memory %llu passes %zu intervals %u tiles %u splits %u long %u chunks %llu many %u breaks %lu mended %lu out_of_hops %lu global_words %lu bad %d\n",
         memory, b->passes.size(), p.n_iv, p.n_tiles, p.n_splits, p.n_long, static_cast<unsigned long long>(chunks), p.many, breaks, mended, out_of_hops,
         global_words, any_bad ? 1 : 0);
  mjd_entropy_batch_destroy(b);
  for (void* o : owned) free(o);
  for (mjd_entropy_job& j : jobs) free(j.d_coef);
  for (Image& im : images) free(im.jpg);
  return rc;
}
