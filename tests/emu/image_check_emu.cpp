// CPU run of the checks of a loaded image (the library's image_check.h): the header checks, the check that
// the device runs on the sections, thread by thread and with every read counted and its index checked, and
// the host's check of the same words.
//
// Usage: image_check_emu THREADS IMAGE UPLOADED: IMAGE holds the words as first read (whose header is
// checked), UPLOADED those that reached the device.  Prints: header accepted, sections fit, device verdict
// (0: accepted), host accepts the uploaded words under the checked header, most reads of one thread, all
// reads, reads out of range, whether a load has the device check the sections.
#include <hip/hip_runtime.h>

#include "image_check.h"

namespace phobic {
void set_error(const std::string&) {}
phobic_status fail(phobic_status s, const std::string&) { return s; }
uint64_t num_partitions(uint64_t n, uint32_t P) { return n ? (n + P - 1) / P : 1; }
}  // namespace phobic

EmuIdx threadIdx, blockIdx, blockDim, gridDim;
EmuWave* emu_wave;

using namespace phobic;

struct Counted {
  const std::vector<uint64_t>* v;
  uint64_t *reads, *outside;
  uint64_t operator[](uint64_t i) const {
    ++*reads;
    if (i < v->size()) return (*v)[i];
    ++*outside;
    return 0;
  }
};

static std::vector<uint64_t> load(const char* path) {
  FILE* f = std::fopen(path, "rb");
  if (!f) std::exit(3);
  std::fseek(f, 0, SEEK_END);
  std::vector<uint64_t> v((size_t)std::ftell(f) / 8);
  std::rewind(f);
  if (std::fread(v.data(), 8, v.size(), f) != v.size()) std::exit(3);
  std::fclose(f);
  return v;
}

int main(int argc, char** argv) {
  if (argc != 4) return 2;
  const uint64_t nt = std::strtoull(argv[1], nullptr, 10);
  const std::vector<uint64_t> first = load(argv[2]);
  std::vector<uint64_t> up = load(argv[3]);
  if (first.size() != up.size() || up.size() < kHeaderWords) return 3;
  ImageHeader h;
  std::memcpy(h.w, first.data(), sizeof(h.w));
  const bool header = check_header(h.w, up.size()) == PHOBIC_OK;
  const bool fit = header && sections_fit(h.w, up.size());
  uint64_t most = 0, all = 0, outside = 0;
  uint32_t bad = 0;
  bool host = false;
  if (fit) {
    for (uint64_t t = 0; t < nt; t++) {
      uint64_t reads = 0;
      bad |= check_part(Counted{&up, &reads, &outside}, h, t, nt);
      most = std::max(most, reads);
      all += reads;
    }
    std::memcpy(up.data(), h.w, sizeof(h.w));
    host = check_sections(up.data(), up.size()) == PHOBIC_OK;
  }
  std::printf("%d %d %u %d %llu %llu %llu %d\n", (int)header, (int)fit, bad, (int)host, (unsigned long long)most,
              (unsigned long long)all, (unsigned long long)outside,
              (int)(header && check_on_device(h.w, up.size())));
  return 0;
}
