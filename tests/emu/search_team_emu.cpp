// CPU run of the team search (search_team of the library's search_team.h) on one partition: W
// wavefronts of 64 coroutines each on one host thread.  A wavefront runs up to its lanes' next
// collective, then a pseudo-random other one is resumed (SEED picks the order), so the wavefronts
// interleave; the workgroup barrier holds every lane until all have reached it.  Built with
// AddressSanitizer over an LDS block of exactly the size the library gives the team.
//
// Usage: search_team_emu WAVES SEED IN OUT; an odd SEED also picks the variant for many pilots per bucket (IN and OUT as in search_emu.cpp)
#include <hip/hip_runtime.h>

void emu_team_barrier();
#define __syncthreads emu_team_barrier
#include SEARCH_SRC

#include <vector>

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

namespace {
SearchArgs g_sa;
uint32_t *g_lds, g_W;
bool g_many;  // odd SEED: the variant for many pilots per bucket
bool g_done[1024];
unsigned g_epoch[1024], g_released;

void lane_main() {
  const unsigned me = threadIdx.x;
  if (g_sa.max_m <= kTeamScratchBits && g_many)
    search_team<true, true, true>(g_sa, 0, g_lds, me >> 6, me & 63, g_W);
  else if (g_sa.max_m <= kTeamScratchBits)
    search_team<true, true, false>(g_sa, 0, g_lds, me >> 6, me & 63, g_W);
  else if (g_sa.max_m < kTeamShiftSlots)
    search_team<true, false, false>(g_sa, 0, g_lds, me >> 6, me & 63, g_W);
  else
    search_team<false, false, false>(g_sa, 0, g_lds, me >> 6, me & 63, g_W);
  g_done[me] = true;
}
}  // namespace

void emu_team_barrier() {
  const unsigned me = threadIdx.x, mine = ++g_epoch[me];
  while (g_released < mine) emu_sync();
}

int main(int argc, char** argv) {
  if (argc != 5) return 2;
  g_W = (uint32_t)std::atoi(argv[1]);
  uint64_t rng = std::strtoull(argv[2], nullptr, 10) * 0x9E3779B97F4A7C15ULL + 1;
  g_many = (std::atoi(argv[2]) & 1) != 0;
  FILE* f = std::fopen(argv[3], "rb");
  uint64_t h[5];
  if (!f || std::fread(h, 8, 5, f) != 5) return 3;
  const uint32_t m = (uint32_t)h[0], B = (uint32_t)h[2];
  const uint64_t limit = h[1], nj = h[3], nb = h[4];
  std::vector<uint64_t> fp(nj);
  std::vector<uint32_t> blist(B, 0);
  if (std::fread(fp.data(), 8, nj, f) != nj || std::fread(blist.data(), 4, nb, f) != nb) return 3;
  std::fclose(f);
  uint32_t maxb = 1;
  for (uint64_t i = 0; i < nb; i++) maxb = std::max<uint32_t>(maxb, blist[i] >> 16);
  std::vector<uint64_t> off = {0, nj}, toff = {0, m};
  std::vector<uint32_t> nbk = {(uint32_t)nb};
  std::vector<uint32_t> pilots(B, 0xDEADBEEFu);
  std::vector<uint32_t> err(1, 0);
  SearchArgs& sa = g_sa;
  sa = SearchArgs{};
  sa.fp = fp.data();
  sa.off = off.data();
  sa.toff = toff.data();
  sa.blist = blist.data();
  sa.nbk = nbk.data();
  sa.pilots = pilots.data();
  sa.err = err.data();
  sa.K = 1;
  sa.limit = limit;
  sa.B = B;
  size_search_lds(sa, std::max<uint32_t>(m, 1), maxb, B, B > 2048);
  const size_t lds = size_team_lds(sa, g_W);
  g_lds = (uint32_t*)std::aligned_alloc(16, lds);
  std::memset(g_lds, 0xA5, lds);  // LDS starts with garbage

  std::vector<EmuWave> waves(g_W);
  constexpr size_t kStack = 1 << 16;
  std::vector<char> stacks(64 * kStack * g_W);
  for (unsigned t = 0; t < 64 * g_W; t++) {
    EmuWave& w = waves[t >> 6];
    const unsigned l = t & 63;
    getcontext(&w.lane[l]);
    w.lane[l].uc_stack.ss_sp = stacks.data() + (size_t)t * kStack;
    w.lane[l].uc_stack.ss_size = kStack;
    w.lane[l].uc_link = &w.sched;
    makecontext(&w.lane[l], lane_main, 0);
  }
  unsigned live = g_W;
  while (live) {
    // barrier: released once every lane has reached it; a wavefront that ended never comes
    unsigned at = 0;
    for (unsigned t = 0; t < 64 * g_W; t++) at += g_epoch[t] == g_released + 1;
    if (at == 64 * g_W) g_released++;
    rng ^= rng << 13;
    rng ^= rng >> 7;
    rng ^= rng << 17;
    const unsigned w = (unsigned)(rng >> 33) % g_W;
    if (g_done[w * 64]) continue;
    const bool waiting = g_epoch[w * 64] > g_released;
    if (waiting) {
      bool others = false;  // somebody must still be able to move
      for (unsigned v = 0; v < g_W; v++) others |= !g_done[v * 64] && g_epoch[v * 64] <= g_released;
      if (!others && at != 64 * g_W) {
        std::fprintf(stderr, "wavefronts left the kernel before a barrier the others wait at\n");
        return 5;
      }
      continue;
    }
    emu_wave = &waves[w];
    const unsigned steps = 1 + (unsigned)(rng >> 20) % 64;  // collectives before another wavefront runs
    for (unsigned q = 0; q < steps && !g_done[w * 64] && g_epoch[w * 64] <= g_released; q++) {
      unsigned now = 0;
      for (unsigned l = 0; l < 64; l++) {
        threadIdx.x = w * 64 + l;
        swapcontext(&waves[w].sched, &waves[w].lane[l]);
        now += g_done[w * 64 + l];
      }
      if (now == 64) {
        live--;
      } else if (now) {
        std::fprintf(stderr, "lanes left the kernel at different collectives\n");
        return 4;
      }
    }
  }
  std::free(g_lds);
  FILE* o = std::fopen(argv[4], "wb");
  std::fwrite(pilots.data(), 4, B, o);
  std::fwrite(err.data(), 4, 1, o);
  std::fclose(o);
  return 0;
}
