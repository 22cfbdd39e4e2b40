// Checks that a serialized image is internally consistent, so the query kernels never read outside it: its
// header and section extents (check_header), then everything in the sections, on the host (check_sections)
// or, for the uploaded image, on the device (check_part).  Part of api.hip; the CPU tests include it too.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>
#include <vector>

#include "phobic_internal.h"

namespace phobic {

inline uint64_t host_bits(const uint64_t* w, uint64_t pos, uint32_t width) {
  if (width == 0) return 0;
  uint64_t idx = pos >> 6;
  uint32_t sh = (uint32_t)(pos & 63);
  uint64_t v = w[idx] >> sh;
  if (sh + width > 64) v |= w[idx + 1] << (64 - sh);
  return width == 64 ? v : (v & ((1ULL << width) - 1));
}

inline uint32_t host_bit_length(uint64_t v) { return v ? 64 - __builtin_clzll(v) : 0; }

inline phobic_status bad_image(const char* what) {
  return fail(PHOBIC_E_FORMAT, std::string("malformed image: ") + what);
}

inline phobic_status check_header(const uint64_t* w, uint64_t nwords) {
  auto bad = bad_image;
  if (nwords < kHeaderWords || w[kHMagic] != kMagic) return bad("magic");
  if (w[kHWords] != nwords) return bad("length");
  const uint64_t n = w[kHN], K = w[kHK], B = w[kHB], total = w[kHTotal];
  const uint64_t coding = w[kHCoding] & 0xFF, bfn = w[kHCoding] >> 8;
  if (K == 0 || B == 0 || B > 65535 || coding > 1 || bfn > PHOBIC_BF_UNIFORM || total < n) return bad("sizes");
  const uint64_t c = w[kHNcompact];  // Compact encoders before the Rice ones (Rice images only)
  if (c > B || (coding != PHOBIC_IC_RICE && c != 0)) return bad("mixed coding");
  const uint32_t an = (uint32_t)w[kHAlpha], ad = (uint32_t)(w[kHAlpha] >> 32);
  if (an == 0 || ad == 0 || an > ad || w[kHP] == 0 || w[kHP] > 0xFFFFFFFFULL) return bad("parameters");
  double lambda;
  std::memcpy(&lambda, &w[kHLambda], 8);
  if (!(lambda > 0.0) || !std::isfinite(lambda) || (uint64_t)std::ceil((double)w[kHP] / lambda) != B)
    return bad("lambda");
  if (K != num_partitions(n, (uint32_t)w[kHP])) return bad("partition count");
  if (w[kHWoff] > 64 || w[kHWremap] > 64) return bad("widths");
  const uint64_t so = w[kHSecOff], se = w[kHSecEnc], sd = w[kHSecData], su = w[kHSecUnary], ss = w[kHSecSel],
                 sr = w[kHSecRemap];
  if (so != kHeaderWords) return bad("section order");
  if (se != so + ((K + 1) * w[kHWoff] + 63) / 64 + 1 || sd != se + B + 1 || su < sd || ss < su || sr < ss ||
      sr > nwords)
    return bad("section layout");
  return PHOBIC_OK;
}

inline phobic_status check_sections(const uint64_t* w, uint64_t nwords) {
  auto bad = bad_image;
  const uint64_t n = w[kHN], K = w[kHK], B = w[kHB], total = w[kHTotal], c = w[kHNcompact];
  const uint64_t coding = w[kHCoding] & 0xFF;
  const uint64_t so = w[kHSecOff], se = w[kHSecEnc], sd = w[kHSecData], su = w[kHSecUnary], ss = w[kHSecSel],
                 sr = w[kHSecRemap];
  // offsets: 0 first, total last, non-decreasing
  uint64_t prev = 0;
  for (uint64_t j = 0; j <= K; j++) {
    uint64_t o = expected_offset_host(j, w[kHR]) + w[kHDmin] + host_bits(w + so, j * w[kHWoff], (uint32_t)w[kHWoff]);
    if ((j == 0 && o != 0) || o < prev || (j == K && o != total)) return bad("offsets");
    prev = o;
  }
  // encoders: payload inside the data section
  const uint64_t data_bits = (su - sd - 1) * 64;
  for (uint64_t i = 0; i < B; i++) {
    const uint64_t e = w[se + i];
    const uint32_t wd = (uint32_t)(e & 0xFF);
    if (wd > 32 || (e >> 8) + (uint64_t)wd * K > data_bits) return bad("encoder table");
  }
  const uint64_t nvals = K * (B - c);  // values of the Rice encoders: one one each in the unary stream
  if (coding == PHOBIC_IC_RICE) {
    const uint64_t ubits = w[kHUbits];
    if (su + (ubits + 63) / 64 + 1 != ss) return bad("unary length");
    uint64_t ones = 0;
    for (uint64_t i = 0; i < (ubits + 63) / 64; i++) ones += __builtin_popcountll(w[su + i]);
    if (ones != nvals || w[ss - 1] != 0) return bad("unary stream");
    const uint64_t nsel = (nvals + kSelBlock - 1) / kSelBlock;
    if (ss + nsel + 1 != sr) return bad("select length");
    // every entry must hold exactly the position of one number kSelBlock s and the distances to ones
    // kSelBlock s + kSelSub k: positions of every kSelSub-th one first
    std::vector<uint64_t> p64((nvals + kSelSub - 1) / kSelSub);
    uint64_t seen = 0, s_next = 0;
    for (uint64_t i = 0; i < (ubits + 63) / 64 && s_next < p64.size(); i++) {
      uint64_t x = w[su + i];
      while (x && s_next < p64.size()) {
        const uint64_t c = (uint64_t)__builtin_popcountll(x);
        const uint64_t want = s_next * kSelSub;
        if (seen + c <= want) {
          seen += c;
          break;
        }
        for (uint64_t skip = want - seen; skip; skip--) x &= x - 1;  // drop ones before the target
        p64[s_next++] = i * 64 + (uint64_t)__builtin_ctzll(x);
        seen = want + 1;
        x &= x - 1;
      }
    }
    if (s_next != p64.size()) return bad("select samples");
    constexpr uint32_t per = kSelBlock / kSelSub;
    for (uint64_t sb = 0; sb < nsel; sb++) {
      const uint64_t a0 = p64[sb * per];
      if (a0 >> 32) return bad("select range");
      uint64_t want = a0;
      for (uint32_t k = 1; k < per; k++) {
        const uint64_t idx = sb * per + k;
        const uint64_t rel = idx < p64.size() ? std::min<uint64_t>(p64[idx] - a0, kSelRelNone) : 0;
        want |= rel << (32 + 10 * (k - 1));
      }
      if (w[ss + sb] != want) return bad("select samples");
    }
  } else if (su != ss || ss != sr) {
    return bad("compact layout");
  }
  const uint64_t nremap = total - n;
  if (w[kHNremap] != nremap || (nremap && w[kHWremap] != (n > 1 ? host_bit_length(n - 1) : 0)))
    return bad("remap");
  const uint64_t want_end = sr + (nremap ? (nremap * w[kHWremap] + 63) / 64 + 1 : 0);
  if (want_end != nwords) return bad("remap length");
  for (uint64_t g = 0; g < nremap; g++)
    if (host_bits(w + sr, g * w[kHWremap], (uint32_t)w[kHWremap]) >= n) return bad("remap entries");
  return PHOBIC_OK;
}

// The same checks on the device, thread tid of nt: returns whether it does not accept what it read.  The
// header h is the one that check_header and sections_fit have passed, never the uploaded words: the caller's
// memory may have changed between the two reads of it.  The select entries are checked segment by segment: entry s names a set bit with exactly
// kSelBlock ones from there to the next entry's (the last one: the remaining ones to the end), and none
// precede entry 0's, so by induction every entry names the one it should; the three distances follow from
// the ones after it.  A thread reads at most kSegmentWords words of a segment, so that entries out of order or
// a stream with long gaps do not make a few threads read the whole stream: what it does not accept, the host
// decides (256 ones of a Rice stream take 12 words on average).  Bound: one pass over the image (0.25 B per key).
constexpr uint64_t kSegmentWords = 256;
struct ImageHeader {
  uint64_t w[kHeaderWords];
};

// width <= 64 bits at bit pos of the section that starts at word `sec`
template <typename Words>
__device__ __forceinline__ uint64_t section_bits(const Words& w, uint64_t sec, uint64_t pos, uint32_t width) {
  if (width == 0) return 0;
  const uint64_t idx = sec + (pos >> 6);
  const uint32_t sh = (uint32_t)(pos & 63);
  uint64_t v = w[idx] >> sh;
  if (sh + width > 64) v |= w[idx + 1] << (64 - sh);
  return width == 64 ? v : (v & ((1ULL << width) - 1));
}

template <typename Words>
__device__ __forceinline__ bool check_part(const Words& w, const ImageHeader& h, uint64_t tid, uint64_t nt) {
  const uint64_t n = h.w[kHN], K = h.w[kHK], B = h.w[kHB], total = h.w[kHTotal], R = h.w[kHR], dmin = h.w[kHDmin];
  const uint64_t sd = h.w[kHSecData], su = h.w[kHSecUnary], ss = h.w[kHSecSel];
  const uint32_t woff = (uint32_t)h.w[kHWoff];
  bool bad = false;
  for (uint64_t j = tid; j <= K; j += nt) {
    const uint64_t o = expected_offset(j, R) + dmin + section_bits(w, h.w[kHSecOff], j * woff, woff);
    if (j == 0 ? o != 0
               : o < expected_offset(j - 1, R) + dmin + section_bits(w, h.w[kHSecOff], (j - 1) * woff, woff))
      bad = true;
    if (j == K && o != total) bad = true;
  }
  const uint64_t data_bits = (su - sd - 1) * 64;
  for (uint64_t i = tid; i < B; i += nt) {
    const uint64_t e = w[h.w[kHSecEnc] + i];
    const uint32_t wd = (uint32_t)(e & 0xFF);
    if (wd > 32 || (e >> 8) + (uint64_t)wd * K > data_bits) bad = true;
  }
  if ((h.w[kHCoding] & 0xFF) == PHOBIC_IC_RICE) {
    const uint64_t nvals = K * (B - h.w[kHNcompact]), nsel = (nvals + kSelBlock - 1) / kSelBlock;
    const uint64_t U = (h.w[kHUbits] + 63) / 64, ubits = U * 64;
    if (tid == 0 && w[su + U] != 0) bad = true;
    if (nsel == 0)
      for (uint64_t x = tid; x < U; x += nt)
        if (w[su + x]) bad = true;
    for (uint64_t s = tid; s < nsel; s += nt) {
      const uint64_t entry = w[ss + s], a = entry & 0xFFFFFFFFULL;
      const uint64_t end = s + 1 < nsel ? w[ss + s + 1] & 0xFFFFFFFFULL : ubits;
      const uint64_t want = s + 1 < nsel ? kSelBlock : nvals - s * kSelBlock;
      if (a >= ubits || end <= a || end > ubits || ((end - 1) >> 6) - (a >> 6) >= kSegmentWords ||
          (s == 0 && a >> 6 >= kSegmentWords) || !((w[su + (a >> 6)] >> (a & 63)) & 1)) {
        bad = true;
        continue;
      }
      if (s == 0) {
        uint64_t before = w[su + (a >> 6)] & ((1ULL << (a & 63)) - 1);
        for (uint64_t x = 0; x < a >> 6; x++) before |= w[su + x];
        if (before) bad = true;
      }
      uint64_t word = a >> 6, x = w[su + word] & (~0ULL << (a & 63)), seen = 0, out = a;
      uint32_t k = 1;  // the next distance: one number kSelSub k from the entry's on
      for (;; x = w[su + ++word]) {
        const bool last = word == (end - 1) >> 6;
        if (last && (end & 63)) x &= (1ULL << (end & 63)) - 1;
        const uint32_t c = __popcll(x);
        for (; k < kSelBlock / kSelSub && k * kSelSub < want && seen + c > k * kSelSub; k++) {
          const uint64_t rel = word * 64 + select_in_word(x, (uint32_t)(k * kSelSub - seen)) - a;
          out |= (rel < kSelRelNone ? rel : kSelRelNone) << (32 + 10 * (k - 1));
        }
        seen += c;
        if (last || seen > want) break;
      }
      if (seen != want) bad = true;
      if (out != entry) bad = true;
    }
  }
  const uint64_t nremap = total - n;
  const uint32_t wr = (uint32_t)h.w[kHWremap];
  for (uint64_t g = tid; g < nremap; g += nt)
    if (section_bits(w, h.w[kHSecRemap], g * wr, wr) >= n) bad = true;
  return bad;
}

// Whether the sections of a checked header lie inside the image, each with its pad word, in arithmetic
// that cannot wrap: what the device check reads.  (The host check refuses what does not fit.)
inline bool sections_fit(const uint64_t* w, uint64_t nwords) {
  const uint64_t K = w[kHK], B = w[kHB], nremap = w[kHTotal] - w[kHN];
  const uint64_t su = w[kHSecUnary], ss = w[kHSecSel], sr = w[kHSecRemap], bits = nwords * 64;
  if (K >> 31 || w[kHUbits] > bits || (K + 1) * w[kHWoff] > bits || su <= w[kHSecData]) return false;
  if (w[kHNremap] != nremap || (nremap && w[kHWremap] != host_bit_length(w[kHN] ? w[kHN] - 1 : 0))) return false;
  if (nremap && (w[kHWremap] == 0 || nremap > bits / w[kHWremap])) return false;
  if (sr + (nremap ? (nremap * w[kHWremap] + 63) / 64 + 1 : 0) != nwords) return false;
  if ((w[kHCoding] & 0xFF) != PHOBIC_IC_RICE) return su == ss && ss == sr;
  return su + (w[kHUbits] + 63) / 64 + 1 == ss &&
         ss + (K * (B - w[kHNcompact]) + kSelBlock - 1) / kSelBlock + 1 == sr;
}

// Whether the sections of an image are checked on the device rather than on the host: a second launch and the
// wait for its answer cost 12 to 20 us a load, so the host keeps the check while it takes less.  It takes
// about 0.15 ns per value of the Rice encoders (the unary stream and its select entries; Compact images have
// neither), 0.6 ns per remap entry, 1 ns per offset and encoder word and 0.07 ns per word of its copy, and
// from 2^17 words on the copy alone (pages mapped anew) costs as much as the device's check.  A load and its
// first 1000 lookups, us, host / device:
//   Rice, lambda 7: 14 571 words 58 / 69, 28 719 77 / 75, 57 090 110 / 85, 284 010 621 / 158
//   Rice, lambda 5: 9914 55 / 68, 16 153 62 / 69, 31 829 85 / 74, 63 091 126 / 84
//   Compact, lambda 7: 10 018 45 / 64, 33 517 58 / 69, 67 573 71 / 81, 136 411 145 / 121, 345 386 234 / 157
//   300 of 358 encoders Compact: 32 544 59 / 75, 65 487 78 / 84, 131 883 158 / 125
//   Compact, alpha 0.9: 11 884 57 / 63, 18 233 67 / 64, 30 363 84 / 68; alpha 0.99: 35 635 62 / 70, 72 171 86 / 81
inline bool check_on_device(const uint64_t* w, uint64_t nwords) {
  if (!sections_fit(w, nwords)) return false;
  const uint64_t rice = (w[kHCoding] & 0xFF) == PHOBIC_IC_RICE ? w[kHK] * (w[kHB] - w[kHNcompact]) : 0;
  const double host_ns = 0.15 * (double)rice + 0.6 * (double)(w[kHTotal] - w[kHN]) + (double)(w[kHK] + w[kHB]) +
                         0.07 * (double)nwords;
  return nwords >= 1 << 17 || host_ns > 17000;
}

}  // namespace phobic
