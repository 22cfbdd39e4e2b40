// CPU run of the search's launch rule: wavefronts per partition for each line "P K lambda b load" of the
// input, K partitions of P keys and largest buckets of b keys on average, `load` with those of other builds, on a device of 256 compute units with 160 KB of LDS.
#include <hip/hip_runtime.h>

#include SEARCH_SRC

namespace phobic {
namespace {
alignas(16) uint32_t lds32[4];
}  // namespace
void set_error(const std::string&) {}
phobic_status fail(phobic_status s, const std::string&) { return s; }
}  // namespace phobic

EmuIdx threadIdx, blockIdx, blockDim, gridDim;
EmuWave* emu_wave;

using namespace phobic;

int main() {
  double P, K, lambda, b, load;
  while (std::scanf("%lf %lf %lf %lf %lf", &P, &K, &lambda, &b, &load) == 5) {
    SearchArgs sa{};
    sa.B = (uint32_t)std::ceil(P / lambda);
    sa.cus = 256;
    sa.lds_limit = 160 * 1024;
    sa.bucket_keys = (float)(P / sa.B);
    sa.load = (uint64_t)load;
    const uint32_t m = (uint32_t)std::ceil(P + 7 * std::sqrt(P) + 16);
    size_search_lds(sa, m, (uint32_t)(b + 7 * std::sqrt(b) + 16), sa.B, m > 8192);
    std::printf("%u\n", team_size(sa, (uint64_t)K, search_config()));
  }
}
