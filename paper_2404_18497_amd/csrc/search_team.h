// Pilot search of one partition by a team of wavefronts (one workgroup); part of search.hip, which
// includes it after its own helpers.
//
// A launch with fewer partitions than the device has wavefront slots (8192) leaves the rest of the
// device idle when one wavefront searches a partition: a partition is a serial chain over its
// buckets.  What makes the chain divisible is that slots are only ever taken: a pilot that was
// rejected for a bucket while fewer slots were taken stays rejected.  So the W wavefronts of a team
// search the next W buckets at the same time, against the table as it is, and in rounds:
//
//   work      a wavefront whose candidate has lost a slot, or that has none, tests one unit of its
//             bucket's pilots (in pilot order) and keeps the first that fits.  One that still holds a
//             candidate, or has no bucket, takes a further unit of the first uncommitted bucket if
//             that had none (units are handed out by a ticket; the lowest pilot found counts; kMany
//             hands out single parts, also to those that found their candidate meanwhile).  Every
//             candidate claims its slots in `claims` (the smallest claim wins: the later round, then
//             the earlier bucket).
//   check     in the run of buckets from the first uncommitted one on that hold a candidate, the
//             first whose slots an earlier bucket claimed too ends the run.
//   commit    the buckets of the run mark their slots and write their pilots, and their wavefronts
//             move on to the buckets W further on.
//
// The first uncommitted bucket's candidate is the smallest pilot that fits the table its predecessors
// left, and so is that of every bucket committed with it (their slots do not meet), which is what the
// sequential search finds.  A candidate that lost its slots goes on from its own unit.  All waits are
// workgroup barriers: one per round, three where a run commits.  The buckets of one key at the end,
// which would meet each other's slots all the time, are placed by one wavefront in a walk over the
// free slots that are left (singles).
//
// Bound: latency (520 partitions at lambda 7: VALU busy 25% of the launch, SALU 33%).  By cycle counters in
// a timed copy, at lambda 7 that of a round (about 6500 cycles, 3.7 buckets committed, of which 4200
// the longest unit of its eight wavefronts and 2300 claims, checks and marks); at lambda 12 the
// parts' chains of LDS round trips (2100 cycles each, whatever the number of wavefronts) and the wait
// for bucket r's.  One partition of 2500 keys: 449 -> 223 us at lambda 7, 15.6 -> 1.95 ms at lambda
// 12; the times over partition counts stand at team_waves.

constexpr uint32_t kTeamPacked = 32;  // buckets up to this size: several seeds per hash evaluation
constexpr uint32_t kTeamPart = 128;   // displacement windows per part of such a bucket's pilots
static_assert(kTeamPart * 64 == kTeamScratchBits, "kFew: whole seeds per part and an exact scratch");

// Inclusive prefix sum over the wavefront: six DPP adds (rows of 16 by shifts, then broadcasts of the rows'
// last lanes), where shuffles would be six LDS round trips.
__device__ __forceinline__ uint32_t wave_prefix(uint32_t v, uint32_t lane) {
#ifdef __HIP__
  (void)lane;
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, true);   // row_shr:1
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, true);   // row_shr:2
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, true);   // row_shr:4
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, true);   // row_shr:8
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);  // row_bcast:15 to rows 1, 3
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);  // row_bcast:31 to rows 2, 3
#else  // the host emulation of the search
  for (uint32_t d = 1; d < 64; d <<= 1) {
    const uint32_t y = __shfl(v, (int)(lane - d) & 63);
    if (lane >= d) v += y;
  }
#endif
  return v;
}

__device__ __forceinline__ void team_failure(const SearchArgs& a, uint64_t j, uint32_t status) {
  atomicOr(a.err, 1u << status);
  if (a.fail_part) atomicMin(a.fail_part, (unsigned long long)j);
}

// Words that one wavefront writes and others read between two barriers (the help protocol of kMany).  The
// waiting loop reads nothing else, so only an atomic read obliges the compiler to read again; release and
// acquire order the words that `state` publishes.  (The host emulation has one thread, whose wavefronts
// change at collectives.)
__device__ __forceinline__ uint32_t shared_acquire(const uint32_t* p) {
#ifdef __HIP__
  return __hip_atomic_load(p, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP);
#else
  return *p;
#endif
}
__device__ __forceinline__ unsigned long long shared_read(const unsigned long long* p) {
#ifdef __HIP__
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
#else
  return *p;
#endif
}
__device__ __forceinline__ void shared_release(uint32_t* p, uint32_t v) {
#ifdef __HIP__
  __hip_atomic_store(p, v, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
#else
  *p = v;
#endif
}

// Places every bucket of partition j; all W wavefronts (a power of two, at most kTeamMaxWaves) call it.
// kShift: F2 has its shifted copy (position codes then hold slots below kTeamShiftSlots).
// kFew: every table of the launch has at most kTeamScratchBits slots, so that a part of a packed bucket's
// pilots is a number of whole seeds and the repeat scratch holds a bit per slot.
// kMany: buckets try many pilots (lambda 9 and more): idle wavefronts help with bucket r, and a part's
// two windows per lane go through the keys together, at 104 registers in place of 77.
template <bool kShift, bool kFew, bool kMany>
__device__ __forceinline__ void search_team(const SearchArgs& a, const uint64_t j, uint32_t* const lds,
                                            const uint32_t wave, const uint32_t lane, const uint32_t W) {
  constexpr unsigned long long kNone = ~0ULL;
  typedef unsigned long long u64;
  // control words: what every wavefront posted in this round and the last one (o, entry, next part,
  // holds a candidate | failures); then per round modulo 3 (a round's set is cleared in the round before
  // it) the helpers' best (pilot << 32 | part), the helpers' tickets, the first bucket of the run that may
  // not commit and, for kMany, the state of bucket r and its place, entry and first part for helpers; then
  // a flag for equal fingerprints and the counts of big buckets and of those with two keys or more
  uint32_t* const post = lds;
  u64* const best = (u64*)(lds + 8 * kTeamMaxWaves);
  uint32_t* const ticket = lds + 8 * kTeamMaxWaves + 6;
  uint32_t* const conflict = ticket + 3;
  uint32_t* const state = conflict + 3;
  uint32_t* const wanted = state + 3;
  uint32_t* const dupflag = wanted + 9;
  uint32_t* const counts = dupflag + 1;
  static_assert(8 * kTeamMaxWaves + 6 + 9 + 9 + 3 <= kTeamCtlWords, "control words");
  enum : uint32_t { kUndecided, kWanted, kDone };  // bucket r in a round: help wanted, or no new parts
  uint32_t* const F2 = lds + kTeamCtlWords;
  uint32_t* const F2s = F2 + a.f2_words;  // kShift: F2 shifted by one word
  uint32_t* const claims = F2 + (kShift ? 2 : 1) * a.f2_words;
  uint32_t* const scr = claims + a.own_words + (size_t)wave * (a.team_scr + a.rb_cap);
  uint32_t* const rbuf = scr + a.team_scr;
  const uint32_t omask = a.own_words - 1;
  const PosCode<kShift> pc{4 * a.f2_words};
  const uint32_t B = a.B, tid = wave * 64 + lane, nthreads = W * 64;

  const uint64_t kb = uniform64(a.off[j]);
  const uint32_t m = uniform((uint32_t)(a.toff[j + 1] - a.toff[j])), nj = uniform((uint32_t)(a.off[j + 1] - kb));
  const uint32_t nb = uniform(a.nbk[j]);
  const uint32_t* const gbl = a.blist + j * B;
  if (m > a.max_m || (nb && uniform(gbl[0]) >> 16 > a.max_bucket)) {  // beyond the LDS layout's bounds
    if (tid == 0) team_failure(a, j, kErrResize);
    return;
  }
  uint32_t* prow = a.pilots + j * B;  // one MPHF: row j; several: column j - Kbase_t of MPHF t
  uint64_t pstride = 1;
  if (a.owner) {
    const uint32_t t = uniform(a.owner[j]);
    const uint64_t jb = uniform64(a.Kbase[t]);
    pstride = uniform64(a.Kt[t]);
    prow = a.pilots + (uint64_t)B * jb + (j - jb);
  } else {
    for (uint32_t x = tid; x < B; x += nthreads) prow[x] = 0;  // empty buckets keep pilot 0
  }
  const uint32_t twom = 2 * m;
  auto f2_init = [&](uint32_t w) -> uint32_t {  // word w of F2 with every slot free
    const uint32_t lo = w * 32;
    return lo + 32 <= twom ? 0xFFFFFFFFu : (lo >= twom ? 0u : ((1u << (twom - lo)) - 1u));
  };
  for (uint32_t w = tid; w < a.f2_words; w += nthreads) {
    F2[w] = f2_init(w);
    if (kShift) F2s[w] = f2_init(w + 1);
  }
  for (uint32_t w = tid; w < a.own_words; w += nthreads) claims[w] = ~0u;
  for (uint32_t w = lane; w < a.team_scr; w += 64) scr[w] = 0;
  if (tid < 3) {
    best[tid] = kNone;
    ticket[tid] = 0;
    conflict[tid] = ~0u;
    state[tid] = kUndecided;
  }
  if (tid == 0) {
    *dupflag = 0;
    counts[0] = counts[1] = 0;
  }
  __syncthreads();
  // sizes are non-increasing: nbig big buckets, then packed ones up to ns, then those of one key
  for (uint32_t x = tid; x < nb; x += nthreads) {
    const uint32_t sx = gbl[x] >> 16, sy = x + 1 < nb ? gbl[x + 1] >> 16 : 0u;
    if (sx > kTeamPacked && sy <= kTeamPacked) counts[0] = x + 1;
    if (sx >= 2 && sy < 2) counts[1] = x + 1;
  }
  __syncthreads();
  const uint32_t nbig = uniform(counts[0]), ns = uniform(counts[1]);

  const char* const F2b = (const char*)F2;
  auto window = [&](uint32_t off, uint32_t sh) -> uint64_t {  // as in search_partition
    const char* p = F2b + off;
    uint32_t w0, w1;
    if (kShift) {
      const uint2 q = *(const uint2*)p;
      w0 = q.x;
      w1 = q.y;
    } else {
      w0 = ((const uint32_t*)p)[0];
      w1 = ((const uint32_t*)p)[1];
    }
    const uint32_t w2 = ((const uint32_t*)p)[2];
    return ((uint64_t)__builtin_amdgcn_alignbit(w2, w1, sh) << 32) | __builtin_amdgcn_alignbit(w1, w0, sh);
  };
  auto take_bit = [&](uint32_t t) {  // as in search_partition
    uint32_t* const w = F2 + (t >> 5);
    const uint32_t mask = ~(1u << (t & 31));
    atomicAnd(w, mask);
    if (kShift) atomicAnd(w + (a.f2_words - 1), mask);
  };
  auto is_taken = [&](uint32_t t) -> bool { return ((F2[t >> 5] >> (t & 31)) & 1u) == 0; };
  auto slot_of = [&](uint32_t pos, uint32_t d) -> uint32_t {
    const uint32_t t = pos + d;
    return t >= m ? t - m : t;
  };
  auto win_mask = [&](uint32_t dlo) -> uint64_t {  // the displacements below m of the window at dlo < m
    return m - dlo >= 64 ? ~0ULL : ((1ULL << (m - dlo)) - 1);
  };
  // ANDs the windows of the kN encoded positions at rb into acc, all reads in flight together
  auto and_keys = [&](const uint32_t* rb, uint64_t& acc, uint32_t loff, auto n) {
    constexpr int kN = decltype(n)::value;
    uint32_t ev[kN];
#pragma unroll
    for (int t = 0; t < kN; t += 4) {
      const uint4 e4 = *(const uint4*)(rb + t);
      ev[t] = e4.x;
      ev[t + 1] = e4.y;
      ev[t + 2] = e4.z;
      ev[t + 3] = e4.w;
    }
    uint64_t w[kN];
#pragma unroll
    for (int t = 0; t < kN; t++) w[t] = window((ev[t] >> 16) + loff, ev[t]);
#pragma unroll
    for (int t = 0; t < kN; t++) acc &= w[t];
  };
  // the same for two windows per lane, with a list of positions each
  auto keys_and2 = [&](const uint32_t* const (&rb)[2], uint64_t (&acc)[2], const uint32_t (&loff)[2], auto n) {
    constexpr int kN = decltype(n)::value;
    uint32_t ev[2][kN];
#pragma unroll
    for (int h = 0; h < 2; h++)
#pragma unroll
      for (int t = 0; t < kN; t += 4) {
        const uint4 e4 = *(const uint4*)(rb[h] + t);
        ev[h][t] = e4.x;
        ev[h][t + 1] = e4.y;
        ev[h][t + 2] = e4.z;
        ev[h][t + 3] = e4.w;
      }
    uint64_t w[2][kN];
#pragma unroll
    for (int h = 0; h < 2; h++)
#pragma unroll
      for (int t = 0; t < kN; t++) w[h][t] = window((ev[h][t] >> 16) + loff[h], ev[h][t]);
#pragma unroll
    for (int h = 0; h < 2; h++)
#pragma unroll
      for (int t = 0; t < kN; t++) acc[h] &= w[h][t];
  };
  // ANDs the windows of the szp encoded positions at rb (szp is 4 or a multiple of 8) into acc; the
  // ballot of the lanes with a bit left
  auto keys_and = [&](const uint32_t* rb, uint64_t& acc, uint32_t loff, uint32_t szp) -> uint64_t {
    if (szp == 4) {
      and_keys(rb, acc, loff, std::integral_constant<int, 4>());
      return uniform64(__ballot(acc != 0));
    }
    uint64_t bal;
    uint32_t k = 0;
    do {
      and_keys(rb + k, acc, loff, std::integral_constant<int, 8>());
      bal = uniform64(__ballot(acc != 0));
      k += 8;
    } while (bal != 0 && k < szp);
    return bal;
  };

  // s m > limit exactly when s > smax; dlast: the largest d allowed with s = smax
  const uint32_t smax = uniform(m ? (uint32_t)min<uint64_t>(a.limit / m, 0xFFFFFFFEULL) : 0u);
  const uint32_t dlast = uniform(m ? (uint32_t)(a.limit - (uint64_t)smax * m) : 0u);
  const uint32_t NW = (m + 63) >> 6;  // windows per seed
  const uint32_t lane_q = NW ? lane / NW : 0u, lane_r = lane - lane_q * NW;
  const uint32_t q64 = NW ? 64u / NW : 0u, r64 = 64u - q64 * NW;
  const uint32_t blocks = (NW + kTeamPart - 1) / kTeamPart;                  // !kFew: parts per seed
  constexpr uint32_t smask = kFew ? ~0u : kTeamScratchBits - 1;  // scratch bit of a position

  auto lg_lanes = [](uint32_t sz) -> uint32_t { return sz <= 4 ? 2u : (sz <= 8 ? 3u : (sz <= 16 ? 4u : 5u)); };
  // the lane's fingerprint of a bucket: key (lane mod S), S lanes per seed, of a packed bucket, else
  // key lane; past the bucket its last key
  auto load_f = [&](uint32_t e, uint32_t o) -> uint64_t {
    const uint32_t sz = e >> 16;
    const uint32_t kx = sz <= kTeamPacked ? lane & ((1u << lg_lanes(sz)) - 1) : lane;
    return a.fp[kb + o + min(kx, sz - 1)];
  };
  // lanes < sz (sz <= 64) with a position r that an earlier lane has (exactly those, when the scratch
  // holds a bit per slot; else possibly others, whose scratch bits meet).  Leaves the scratch clear.
  auto marked_before = [&](uint32_t r, uint32_t sz) -> uint64_t {
    const uint32_t ix = r & smask, bit = 1u << (ix & 31);
    bool c = false;
    if (lane < sz) c = (atomicOr(&scr[ix >> 5], bit) & bit) != 0;
    const uint64_t bm = uniform64(__ballot(c));
    if (lane < sz) scr[ix >> 5] = 0;
    wave_sync();
    return bm;
  };
  auto small_repeats = [&](uint32_t r, uint32_t sz) -> bool {
    uint64_t bm = marked_before(r, sz);
    if (kFew) return bm != 0;
    for (; bm; bm &= bm - 1) {
      const uint32_t c = (uint32_t)__builtin_ctzll(bm);
      const uint32_t rc = __builtin_amdgcn_readlane(r, c);
      if (uniform64(__ballot(lane < sz && lane != c && r == rc))) return true;
    }
    return false;
  };
  // whether two keys of a packed bucket share their fingerprint (then they repeat under every seed)
  auto small_dup = [&](uint64_t f, uint32_t sz) -> bool {
    uint64_t bm = marked_before(pos_hash(f, kPhi64, m), sz);
    for (; bm; bm &= bm - 1) {
      const uint32_t c = (uint32_t)__builtin_ctzll(bm);
      const uint64_t fc = lane_value64(f, c);
      if (uniform64(__ballot(lane < sz && lane != c && f == fc))) return true;
    }
    return false;
  };
  // Positions of a big bucket under seed s to rbuf; whether one repeats (seeds past 0 stop at the first
  // group of 64 keys that does; seed 0 goes on and looks for equal fingerprints, dup).
  auto big_repeats = [&](const uint64_t* keys, uint64_t f0, uint32_t sz, uint32_t s, bool& dup) -> bool {
    const uint64_t w = (uint64_t)(s + 1) * kPhi64;
    bool rep = false;
    uint32_t g = 0, r = 0;
    for (; g * 64 < sz; g++) {
      const uint32_t k = g * 64 + lane;
      const uint64_t f = g == 0 ? f0 : keys[min(k, sz - 1)];
      r = pos_hash(f, w, m);
      bool c = false;
      if (k < sz) {
        rbuf[k] = pc.enc(r);
        const uint32_t ix = r & smask, bit = 1u << (ix & 31);
        c = (atomicOr(&scr[ix >> 5], bit) & bit) != 0;
      }
      uint64_t bm = uniform64(__ballot(c));
      wave_sync();
      for (; bm; bm &= bm - 1) {
        const uint32_t cl = (uint32_t)__builtin_ctzll(bm), kc = g * 64 + cl;
        if (!kFew && !rep) {  // the scratch bits met: do the positions?
          const uint32_t ec = rbuf[kc];
          bool hit = false;
          for (uint32_t x = lane; x < kc; x += 64) hit |= rbuf[x] == ec;
          rep = uniform64(__ballot(hit)) != 0;
        } else {
          rep = true;
        }
        if (s == 0) {
          const uint64_t fc = lane_value64(f, cl);
          bool hit = false;
          for (uint32_t x = lane; x < sz; x += 64) hit |= x != kc && keys[x] == fc;
          if (uniform64(__ballot(hit))) dup = true;
        } else if (rep) {
          break;
        }
      }
      if (rep && s != 0) {
        g++;
        break;
      }
    }
    const uint32_t marked = min(g * 64, sz);
    for (uint32_t k = lane; k < marked; k += 64) scr[(pc.dec(rbuf[k]) & smask) >> 5] = 0;
    if (!rep) {
      const uint32_t last = __builtin_amdgcn_readlane(r, (sz - 1) & 63);
      const uint32_t k = sz + lane;
      if (k < ((sz + 7) & ~7u)) rbuf[k] = pc.enc(last);
    }
    wave_sync();
    return rep;
  };
  // displacement scans of the big bucket in rbuf, as in search_partition
  const uint32_t gw = lane & 7, gg = lane >> 3;
  auto scan8 = [&](uint32_t szp8) -> uint32_t {
    uint64_t acc = 64 * gw < m ? win_mask(64 * gw) : 0ULL;
    const uint32_t loff = 64 * gw < m ? gw * 8 : 0u;
    for (uint32_t k = 0;;) {
      const uint32_t e = rbuf[k + gg];
      acc &= window((e >> 16) + loff, e);
      k += 8;
      if (k >= szp8) break;
      const uint64_t b = uniform64(__ballot(acc != 0));
      if (((b - 0x0101010101010101ULL) & ~b & 0x8080808080808080ULL) != 0) return 0xFFFFFFFFu;
    }
    acc &= __shfl_xor(acc, 8);
    acc &= __shfl_xor(acc, 16);
    acc &= __shfl_xor(acc, 32);
    const uint64_t b = uniform64(__ballot(acc != 0)) & 0xFFull;
    if (!b) return 0xFFFFFFFFu;
    const uint32_t L = (uint32_t)__builtin_ctzll(b);
    return L * 64 + (uint32_t)__builtin_ctzll(lane_value64(acc, L));
  };
  auto scan_all = [&](uint32_t szp8) -> uint32_t {
    for (uint32_t d0 = 0; d0 < m; d0 += 4096) {
      const uint32_t dl = d0 + lane * 64;
      uint64_t acc = dl < m ? win_mask(dl) : 0ULL;
      const uint64_t bal = keys_and(rbuf, acc, dl < m ? dl >> 3 : 0u, szp8);
      if (bal) {
        const uint32_t L = (uint32_t)__builtin_ctzll(bal);
        return d0 + L * 64 + (uint32_t)__builtin_ctzll(lane_value64(acc, L));
      }
    }
    return 0xFFFFFFFFu;
  };

  uint32_t fs = 0, fd = 0, fslot = 0;  // a found pilot's seed, displacement and (key lane's) slot
  // Part u of the pilots of a packed bucket (the lane's fingerprint f): the smallest that fits, as
  // (pilot << 32 | u), or kNone.  over: the bucket has no pilot up to the limit if the parts before u
  // hold none.  A part is as many whole seeds as kTeamPart windows and one hash evaluation hold
  // (kFew), else kTeamPart windows of a seed.
  auto packed_part = [&](uint64_t f, uint32_t sz, uint32_t u, bool& over) -> u64 {
    const uint32_t lgS = lg_lanes(sz), S = 1u << lgS;
    const uint32_t nu = kFew ? min(64u >> lgS, max(1u, kTeamPart / NW)) : 1u;
    const uint64_t s064 = kFew ? (uint64_t)u * nu : u / blocks;
    if (s064 > smax) {
      over = true;
      return kNone;
    }
    const uint32_t s0 = (uint32_t)s064;
    const uint32_t w0 = kFew ? 0u : (u - s0 * blocks) * kTeamPart;
    const uint32_t nwin = kFew ? nu * NW : min(kTeamPart, NW - w0);
    rbuf[lane] = pc.enc(pos_hash(f, (uint64_t)(s0 + (kFew ? lane >> lgS : 0u) + 1) * kPhi64, m));
    wave_sync();
    if constexpr (kMany) {
      // Lane x takes windows x and 64 + x of the part, in pilot order over its seeds.  Both go through the
      // keys together, all reads of eight keys in flight: a part is a chain of LDS round trips.
      uint32_t t[2], dw[2];
      uint64_t acc[2], bal[2];
      const uint32_t* rb[2];
      uint32_t loff[2];
#pragma unroll
      for (int h = 0; h < 2; h++) {
        bool act;
        if (kFew) {
          dw[h] = h ? r64 + lane_r : lane_r;
          t[h] = h ? q64 + lane_q : lane_q;
          if (h && dw[h] >= NW) {
            dw[h] -= NW;
            t[h]++;
          }
          act = t[h] < nu && t[h] <= smax - s0;
        } else {
          dw[h] = w0 + 64 * h + lane;
          t[h] = 0;
          act = 64 * h + lane < nwin;
        }
        acc[h] = act ? win_mask(dw[h] * 64) : 0ULL;
        rb[h] = rbuf + (act ? t[h] * S : 0u);
        loff[h] = act ? dw[h] * 8 : 0u;
      }
      if (S == 4) {
        keys_and2(rb, acc, loff, std::integral_constant<int, 4>());
      } else {
        for (uint32_t k = 0;;) {
          keys_and2(rb, acc, loff, std::integral_constant<int, 8>());
          k += 8;
          if (k >= sz || uniform64(__ballot((acc[0] | acc[1]) != 0)) == 0) break;
          rb[0] += 8;
          rb[1] += 8;
        }
      }
#pragma unroll
      for (int h = 0; h < 2; h++) bal[h] = uniform64(__ballot(acc[h] != 0));
#pragma unroll
      for (int h = 0; h < 2; h++) {
        while (bal[h]) {
          const uint32_t L = (uint32_t)__builtin_ctzll(bal[h]);
          const uint32_t tL = __builtin_amdgcn_readlane(t[h], L);
          const uint32_t d =
              64 * __builtin_amdgcn_readlane(dw[h], L) + (uint32_t)__builtin_ctzll(lane_value64(acc[h], L));
          const uint32_t sd = s0 + tL;
          if (sd == smax && d > dlast) {
            over = true;
            return kNone;
          }
          const uint32_t pos = pc.dec(rbuf[tL * S + (lane < sz ? lane : 0u)]);
          if (!small_repeats(pos, sz)) {
            fs = sd;
            fd = d;
            fslot = slot_of(pos, d);
            return ((u64)(sd * m + d) << 32) | u;
          }
          bal[0] &= ~uniform64(__ballot(t[0] == tL));
          bal[1] &= ~uniform64(__ballot(t[1] == tL));
        }
      }
    } else {
      uint32_t t0 = 0, r0 = 0;
      for (uint32_t c = 0; c < nwin; c += 64) {
        uint32_t dw, t;
        bool act;
        if (kFew) {  // lane x of chunk c takes window c + x of the seeds' windows in pilot order
          dw = r0 + lane_r;
          t = t0 + lane_q;
          if (dw >= NW) {
            dw -= NW;
            t++;
          }
          act = t < nu && t <= smax - s0;
        } else {
          dw = w0 + c + lane;
          t = 0;
          act = c + lane < nwin;
        }
        const uint32_t dlo = dw * 64;
        uint64_t acc = act ? win_mask(dlo) : 0ULL;
        uint64_t bal = keys_and(rbuf + (act ? t * S : 0u), acc, act ? dw * 8 : 0u, S > 8 ? (sz + 7) & ~7u : S);
        while (bal) {
          const uint32_t L = (uint32_t)__builtin_ctzll(bal);
          const uint32_t tL = __builtin_amdgcn_readlane(t, L);
          const uint32_t d = __builtin_amdgcn_readlane(dlo, L) + (uint32_t)__builtin_ctzll(lane_value64(acc, L));
          const uint32_t sd = s0 + tL;
          if (sd == smax && d > dlast) {
            over = true;
            return kNone;
          }
          const uint32_t pos = pc.dec(rbuf[tL * S + (lane < sz ? lane : 0u)]);
          if (!small_repeats(pos, sz)) {
            fs = sd;
            fd = d;
            fslot = slot_of(pos, d);
            return ((u64)(sd * m + d) << 32) | u;
          }
          bal &= ~uniform64(__ballot(t == tL));
        }
        if (kFew) {
          t0 += q64;
          r0 += r64;
          if (r0 >= NW) {
            r0 -= NW;
            t0++;
          }
        }
      }
    }
    return kNone;
  };
  // Part u of a big bucket (o keys before it) is seed u; dup: two equal fingerprints
  auto big_part = [&](const uint64_t* keys, uint64_t f, uint32_t sz, uint32_t o, uint32_t u, bool& over,
                      bool& dup) -> u64 {
    if (u > smax) {
      over = true;
      return kNone;
    }
    if (big_repeats(keys, f, sz, u, dup)) return kNone;
    // the short scan first while the bucket expects three admissible displacements below 512
    uint32_t d = 0xFFFFFFFFu;
    if (m > 512 && (float)sz * __logf((float)(m - o) / (float)m) >= -5.14f) d = scan8((sz + 7) & ~7u);
    if (d == 0xFFFFFFFFu) d = scan_all((sz + 7) & ~7u);
    if (d == 0xFFFFFFFFu) return kNone;
    if (u == smax && d > dlast) {
      over = true;
      return kNone;
    }
    fs = u;
    fd = d;
    fslot = slot_of(pc.dec(rbuf[min(lane, sz - 1)]), d);
    return ((u64)(u * m + d) << 32) | u;
  };
  // parts of a unit that starts at part u: more once the first ones held no pilot, so that a round's
  // barriers are paid for less often; of a big bucket several at once, as most seeds repeat a position
  auto unit_parts = [](bool big, uint32_t u) -> uint32_t {
    return big ? (kFew ? 4u : 2u) : (u == 0 ? 1u : (u < 4 ? 2u : (u < 16 ? 4u : 8u)));
  };

  // The buckets of one key, in order (wavefront 0): key i takes the first free slot at or after its
  // position.  The free slots are listed once (in `claims`) and live on as a bitmap over their ranks, a
  // word per lane; a key's first rank comes from a search in the list, 64 keys at a time, and the
  // walk itself only reads lanes.  More free slots than that (non-minimal tables) are scanned.
  auto singles = [&]() {
    const uint32_t q = nb - ns, o1 = nj - q, Q = m - o1;
    const bool listed = Q <= min(a.own_words, 4096u);
    uint64_t alive = 0;
    if (listed) {
      uint32_t base = 0;
      for (uint32_t x0 = 0; x0 * 64 < m; x0 += 64) {
        const uint32_t x = x0 + lane;
        uint64_t v = x * 64 < m ? (((uint64_t)F2[2 * x + 1] << 32) | F2[2 * x]) & win_mask(x * 64) : 0ULL;
        const uint32_t c = (uint32_t)__popcll(v);
        const uint32_t inc = wave_prefix(c, lane);
        for (uint32_t at = base + inc - c; v; v &= v - 1) claims[at++] = x * 64 + (uint32_t)__builtin_ctzll(v);
        base += __builtin_amdgcn_readlane(inc, 63);
      }
      alive = lane * 64 < Q ? (Q - lane * 64 >= 64 ? ~0ULL : (1ULL << (Q - lane * 64)) - 1) : 0ULL;
      wave_sync();
    }
    bool over = false;
    for (uint32_t i0 = 0; i0 < q; i0 += 64) {
      const uint32_t cnt = min(64u, q - i0), i = i0 + min(lane, cnt - 1);
      const uint32_t p = pos_hash(a.fp[kb + o1 + i], kPhi64, m);
      uint32_t slot = 0;
      if (listed) {
        uint32_t lo = 0, hi = Q;  // the first rank whose slot is at or after p
        while (uniform64(__ballot(lo < hi))) {
          const uint32_t mid = min((lo + hi) >> 1, Q - 1);
          const bool below = claims[mid] < p;
          if (lo < hi) {
            if (below) lo = mid + 1; else hi = mid;
          }
        }
        if (lo == Q) lo = 0;
        uint32_t mine = 0;
        for (uint32_t k = 0; k < cnt; k++) {
          const uint32_t rk = __builtin_amdgcn_readlane(lo, k);
          uint32_t x = rk >> 6;
          uint64_t v = lane_value64(alive, x) & (~0ULL << (rk & 63));
          if (v == 0) {
            const uint64_t any = uniform64(__ballot(alive != 0));
            const uint64_t up = x == 63 ? 0 : any & (~0ULL << (x + 1));
            x = (uint32_t)__builtin_ctzll(up ? up : any);
            v = lane_value64(alive, x);
          }
          const uint32_t b = (uint32_t)__builtin_ctzll(v);
          if (lane == x) alive &= ~(1ULL << b);
          if (lane == k) mine = x * 64 + b;
        }
        slot = claims[mine];
      } else {
        for (uint32_t k = 0; k < cnt; k++) {
          const uint32_t pk = __builtin_amdgcn_readlane(p, k);
          if (lane < 4) rbuf[lane] = pc.enc(pk);
          wave_sync();
          const uint32_t t = slot_of(pk, scan_all(4));
          if (lane == 0) {
            take_bit(t);
            take_bit(t + m);
          }
          if (lane == k) slot = t;
          wave_sync();
        }
      }
      const uint32_t d = slot >= p ? slot - p : slot + m - p;
      if (uniform64(__ballot(smax == 0 && lane < cnt && d > dlast))) {
        over = true;
        break;
      }
      if (lane < cnt) {
        prow[(gbl[ns + i] & 0xFFFF) * pstride] = d;
        if (listed) atomicAnd(&F2[slot >> 5], ~(1u << (slot & 31)));  // for the occupancy bitmap
      }
    }
    if (over && lane == 0) team_failure(a, j, PHOBIC_E_PILOT_OVERFLOW);
  };

  // The bucket list in processing order: entries bbase + lane (bw0) and bbase + 64 + lane (bw1), the
  // keys before bbase (obase) and, inside the window, before each entry (px).
  uint32_t bbase = 0, obase = 0, px = 0, tot = 0;
  uint32_t bw0 = lane < nb ? gbl[lane] : 0u, bw1 = 64 + lane < nb ? gbl[64 + lane] : 0u;
  auto prefix = [&]() {
    const uint32_t v = bw0 >> 16, inc = wave_prefix(v, lane);
    px = inc - v;
    tot = __builtin_amdgcn_readlane(inc, 63);
  };
  prefix();
  auto look = [&](uint32_t x, uint32_t& e, uint32_t& o) {  // x never decreases and moves by at most 64
    if (x >= bbase + 64) {
      obase += tot;
      bbase += 64;
      bw0 = bw1;
      bw1 = bbase + 64 + lane < nb ? gbl[bbase + 64 + lane] : 0u;
      prefix();
    }
    e = __builtin_amdgcn_readlane(bw0, x - bbase);
    o = obase + __builtin_amdgcn_readlane(px, x - bbase);
  };
  // this wavefront's bucket idx (entry e, o keys before it, the lane's fingerprint f) and the one W
  // further on, whose fingerprints are in flight meanwhile
  uint32_t idx = wave, e = 0, o = 0, ne = 0, no = 0;
  uint64_t f = 0, nf = 0;
  bool has = false;  // holds a candidate: pilot cp = cs m + cd of part u, slots ct (keys < 64)
  uint32_t u = 0, cp = 0, cs = 0, cd = 0, ct = 0;
  if (idx < ns) {
    look(idx, e, o);
    f = load_f(e, o);
    if (idx + W < ns) {
      look(idx + W, ne, no);
      nf = load_f(ne, no);
    }
  }
  auto advance = [&]() {
    idx += W;
    e = ne;
    o = no;
    f = nf;
    has = false;
    u = 0;
    if (idx + W < ns) {
      look(idx + W, ne, no);
      nf = load_f(ne, no);
    }
  };

  uint32_t r = 0;              // the first uncommitted bucket
  uint32_t par = 0, b3 = 0;    // the round modulo 2 and 3
  uint32_t round = 0, fl = 0;
  // the rounds for the buckets below `limit`, all of them big or all of them packed
  auto rounds = [&](auto big_tag, uint32_t limit) {
    constexpr bool kBig = decltype(big_tag)::value;
    // fn(slot) for every key of the candidate, on some lane; returns whether one returned true
    auto any_slot = [&](auto fn) -> bool {
      const uint32_t sz = e >> 16;
      bool hit = lane < sz && fn(ct);
      if (kBig) {
        for (uint32_t k0 = 64; k0 < sz; k0 += 64) {
          const uint32_t k = k0 + lane;
          if (k < sz) hit |= fn(slot_of(pos_hash(a.fp[kb + o + k], (uint64_t)(cs + 1) * kPhi64, m), cd));
        }
      }
      return uniform64(__ballot(hit)) != 0;
    };
    bool help = false;  // !kMany: bucket r had no candidate after the last round: its next unit starts at hu
    uint32_t hu = 0;
    uint4 pv{0, 0, 0, 0};  // lane x: what wavefront x mod W posted last
    while (r < limit) {
      const uint32_t n3 = b3 == 2 ? 0u : b3 + 1, w0 = r & (W - 1);  // w0: bucket r's wavefront
      if (tid == 0) {
        best[n3] = kNone;
        ticket[n3] = 0;
        conflict[n3] = ~0u;
        state[n3] = kUndecided;
      }
      // ---- work ----
      const bool mine = idx < limit, first = wave == w0;
      const uint32_t order = idx - r;
      const uint32_t claim = ~(round * kTeamMaxWaves + (kTeamMaxWaves - 1 - order));
      if (mine && has && any_slot([&](uint32_t t) { return is_taken(t); })) has = false;
      uint32_t fmark = 0;
      if constexpr (!kMany) {  // help in units, handed out to those that start the round idle
        const bool my_work = mine && !has;
        uint32_t hx = 0;
        if (my_work || help) {
          uint32_t we = e, wo = o, wu = u;
          uint64_t wf = f;
          if (!my_work) {
            uint32_t tk = 0;
            if (lane == 0) tk = atomicAdd(&ticket[b3], 1u);
            wo = __builtin_amdgcn_readlane(pv.x, w0);
            we = __builtin_amdgcn_readlane(pv.y, w0);
            hx = unit_parts(kBig, hu);
            wu = hu + hx * (1 + uniform(tk));
            wf = load_f(we, wo);
          }
          const uint32_t parts = my_work ? unit_parts(kBig, wu) : hx;
          bool over = false, dup = false;
          u64 c = kNone;
          for (uint32_t i = 0; i < parts && c == kNone && !over; i++)
            c = kBig ? big_part(a.fp + kb + wo, wf, we >> 16, wo, wu + i, over, dup)
                     : packed_part(wf, we >> 16, wu + i, over);
          if (!my_work) {
            if (c != kNone && lane == 0) atomicMin(&best[b3], c);
          } else if (c != kNone) {
            has = true;
            u = (uint32_t)c;
            cp = (uint32_t)(c >> 32);
            cs = fs;
            cd = fd;
            ct = fslot;
          } else {
            if (!kBig && u == 0 && small_dup(f, e >> 16)) dup = true;
            u += parts;
            fmark = dup ? 2u : (over ? 4u : 0u);
          }
        }
      } else {  // help in single parts, as long as bucket r's own wavefront has more than one to go
        bool own = mine && !has;
        uint32_t parts = 0;
        if (first) {
          parts = unit_parts(kBig, u);
          // help is wanted until the last part starts: nobody starts one that would end after it
          const bool ask = own && parts > 1;
          if (ask && lane == 0) {
            wanted[3 * b3] = o;
            wanted[3 * b3 + 1] = e;
            wanted[3 * b3 + 2] = u + parts;
          }
          if (lane == 0) shared_release(&state[b3], ask ? kWanted : kDone);
        }
        uint64_t hf = 0;  // the lane's fingerprint of the helped bucket, once loaded
        uint32_t he = 0, ho = 0, hp = 0;
        for (uint32_t left = parts;;) {
          uint32_t we = e, wo = o, wu = u;
          uint64_t wf = f;
          if (!own) {
            if (first) break;
            const uint32_t st = uniform(shared_acquire(&state[b3]));
            if (st == kDone) break;
            if (st == kUndecided) continue;  // bucket r's wavefront decides after one look at its candidate
            if (uniform64(shared_read(&best[b3])) != kNone) break;
            if (he == 0) {
              ho = uniform(wanted[3 * b3]);
              he = uniform(wanted[3 * b3 + 1]);
              hp = uniform(wanted[3 * b3 + 2]);
              hf = load_f(he, ho);
            }
            uint32_t tk = 0;
            if (lane == 0) tk = atomicAdd(&ticket[b3], 1u);
            we = he;
            wo = ho;
            wu = hp + uniform(tk);
            wf = hf;
          }
          bool over = false, dup = false;
          const u64 c = kBig ? big_part(a.fp + kb + wo, wf, we >> 16, wo, wu, over, dup)
                             : packed_part(wf, we >> 16, wu, over);
          if (!own) {
            if (c != kNone && lane == 0) atomicMin(&best[b3], c);
            continue;
          }
          if (c != kNone) {
            has = true;
            cp = (uint32_t)(c >> 32);
            cs = fs;
            cd = fd;
            ct = fslot;
            own = false;
          } else {
            if (!kBig && u == 0 && small_dup(f, e >> 16)) dup = true;
            u++;
            fmark = dup ? 2u : (over ? 4u : 0u);
            if (fmark) break;
            if (first) {
              if (--left == 0) break;
              if (left == 1 && lane == 0) shared_release(&state[b3], kDone);
            } else if (uniform(shared_acquire(&state[b3])) == kDone) {
              break;
            }
          }
        }
        if (first && lane == 0) shared_release(&state[b3], kDone);
      }
      if (mine && has)
        any_slot([&](uint32_t t) {
          atomicMin(&claims[t & omask], claim);
          return false;
        });
      if (lane == 0) {
        uint32_t* const p = post + (par * kTeamMaxWaves + wave) * 4;
        if (!kMany) {
          p[0] = o;
          p[1] = e;
          p[2] = u;
        }
        p[3] = (mine && has ? 1u : 0u) | fmark;
      }
      __syncthreads();
      // ---- check ----
      const uint32_t* const pp = post + (par * kTeamMaxWaves + (lane & (W - 1))) * 4;
      if (kMany)
        pv.w = pp[3];
      else
        pv = *(const uint4*)pp;
      const bool wins =
          mine && order > 0 && has ? !any_slot([&](uint32_t t) { return claims[t & omask] != claim; }) : true;
      if (__ballot(pv.w > 1)) {
        fl = __ballot((pv.w & 2) != 0) ? 1u : 2u;
        return;
      }
      const uint32_t wmask = (1u << W) - 1;
      const uint32_t flags = (uint32_t)uniform64(__ballot(pv.w != 0)) & wmask;
      uint32_t run = ((flags >> w0) | (flags << (W - w0))) & wmask;  // bit i: bucket r + i holds a candidate
      if ((kMany || help) && (run & 1) == 0) {
        const u64 bp = uniform64(best[b3]);
        if (bp != kNone) {  // a helper found bucket r's pilot: it commits alone, as it claimed nothing
          run = 1;
          if (first) {
            has = true;
            cp = (uint32_t)(bp >> 32);
            cs = cp / m;
            cd = cp - cs * m;
            ct = slot_of(pos_hash(f, (uint64_t)(cs + 1) * kPhi64, m), cd);
          }
        }
      }
      uint32_t L = (uint32_t)__builtin_ctz(~run);
      if (L > 1) {
        if (!wins && order < L && lane == 0) atomicMin(&conflict[b3], order);
        __syncthreads();
        L = min(L, uniform(conflict[b3]));
      }
      // ---- commit ----
      if (L) {
        if (mine && order < L) {
          any_slot([&](uint32_t t) {
            take_bit(t);
            take_bit(t + m);
            return false;
          });
          if (lane == 0) prow[(e & 0xFFFF) * pstride] = cp;
          advance();
        }
        r += L;
        if (!kMany) {
          help = false;
          if (L < W && r < limit) {  // the next first bucket, if no candidate was posted for it
            help = __builtin_amdgcn_readlane(pv.w, r & (W - 1)) == 0;
            hu = __builtin_amdgcn_readlane(pv.z, r & (W - 1));
          }
        }
        __syncthreads();
      } else if (kMany) {  // the helpers found none either
        if (first) u += uniform(ticket[b3]);
      } else {
        uint32_t next = __builtin_amdgcn_readlane(pv.z, w0);
        if (help) next += uniform(ticket[b3]) * unit_parts(kBig, hu);
        help = true;
        hu = next;
        if (first) u = hu;
      }
      if (++round == 1u << 24) {  // claims hold 24 bits of the round
        round = 0;
        __syncthreads();
        for (uint32_t w = tid; w < a.own_words; w += nthreads) claims[w] = ~0u;
        __syncthreads();
      }
      par ^= 1;
      b3 = n3;
    }
  };
  rounds(std::true_type(), nbig);
  if (!fl) rounds(std::false_type(), ns);

  if (fl) {  // the partition has failed; equal fingerprints anywhere are reported first
    if (!(fl & 1)) {
      bool dup = false;
      while (idx < ns) {
        if (e >> 16 > kTeamPacked)
          (void)big_repeats(a.fp + kb + o, f, e >> 16, 0, dup);
        else if (small_dup(f, e >> 16))
          dup = true;
        advance();
      }
      if (dup && lane == 0) atomicOr(dupflag, 1u);
      __syncthreads();
      if (uniform(*dupflag)) fl |= 1;
    }
    if (tid == 0) team_failure(a, j, fl & 1 ? PHOBIC_E_DUPLICATE : PHOBIC_E_PILOT_OVERFLOW);
    return;
  }
  if (ns < nb && wave == 0) singles();
  if (a.taken) {
    __syncthreads();
    const uint64_t tb = uniform64(a.toff[j]);
    for (uint32_t w = tid; w * 32 < m; w += nthreads) {
      const uint32_t nbits = min(32u, m - w * 32);
      const uint32_t busy = ~F2[w] & (nbits == 32 ? 0xFFFFFFFFu : ((1u << nbits) - 1));
      put_bits_atomic(a.taken, tb + (uint64_t)w * 32, busy, nbits);
    }
  }
}
