// Logs of kTinyMax / kWalkMax + 1 .. kMidMax records (part of analyze.hip).
//
// Such a log is bound by the number and the latency of its launches, not by its
// bytes: the 79 launches of the pipeline for longer logs took 290 us for 100,000
// records, whose bytes take 2. Random accesses to tables that stay in the caches
// are cheap here (25 G compare-and-swaps a second), so the groups come from hash
// tables, and 13 launches remain, the longest chain 9 (11 with Algorithm 2's
// pairs): 107 us. Where a key is shared by many records, their updates meet in
// few words, so lanes or chunks of one key go to the tables once.
// The last length here is what the fields below hold (owners, chunks and groups
// in 32 bits), not where the sorts become faster: 262,144 records take 130 us
// here, 262,145 take 282 by sorts. (At 10.7 million records the tables' atomics
// would cost 0.4 ms per access to each record, more than the sort passes.)
//
//   clear     the digest table, the call's counters
//   classify  as in the pipeline; each transfer also finds its digest's slot in
//             the table: its group number, exact, so the sort that follows
//             needs two passes over the group number and no fix-up
//   scan      wavefront counts and the classification's sums
//   digest path: two scatters (each sums the tile histograms it needs itself),
//             group aggregates, DD/RT (carries looked up, not scanned)
//   other path: subsets; unused transfers and the groups of ALLOC/DELETE
//             records; pairing and RA table; RA/UA. The nearest record of a
//             group comes from its chunk of the list, grouped in LDS, and the
//             group's table entries per chunk (NearTable) instead of a sort
//   finish    all sums into the report
#pragma once

constexpr uint32_t kMidMax = 262144;
constexpr int kMidT = 1024, kMidRounds = 2;
constexpr uint32_t kMidTile = kMidT * kMidRounds;           // records (elements) per workgroup
constexpr uint32_t kMidWave = 64 * kMidRounds;              // ... per wavefront
constexpr uint32_t kMidDigits = 1024;                       // at most, per pass
constexpr uint32_t kChunkWords = 4;                         // 64 chunks of a NearTable each
constexpr uint32_t kChunkMax = 1024;                        // positions per chunk, at most
static_assert(kChunkWords * 64 * kChunkMax >= kMidMax, "a chunk is one bit of the words");

// Groups of equal keys over a list of positions (0 .. m - 1, m <= kMidMax), and
// the nearest earlier position of a group (REV: of the list read backwards, so
// the nearest later one). A workgroup enters a chunk of the list at a time
// (near_enter): it groups the chunk's positions in LDS, which gives each one's
// neighbour inside the chunk, and then touches the tables once per group and
// chunk only: a position's group is the slot of its key in an open-addressing
// table; per group, a bit for each chunk that holds it; per (group, chunk), the
// last such position. A position whose neighbour lies in an earlier chunk finds
// it by those (near_prev). No step depends on how far apart a group's
// positions are or how many share it. (Entering position by position, with a
// search through the list inside a chunk of 2,048, took 411 us for 262,144
// ALLOC/DELETE records of 10 addresses, all updates going to few words, and
// 454 us when each array is freed 2,000 records after its allocation; by
// chunks 137 and 165 us. 100,000 records of the trace, few of them such: 111
// and 107 us.)
struct NearTable {
  uint32_t* owner;           // group table (below)
  unsigned long long* bits;  // [slots][kChunkWords]
  uint32_t *ckey, *clast;    // 0 empty, else (group << 8 | chunk) + 1; the last position
  uint32_t* link;            // per position: the neighbour in its chunk, else kFar | group
};
constexpr uint32_t kFar = 0x80000000u;
// Positions per chunk: the list in at most kChunkWords * 64 of them, and not
// fewer than a workgroup has threads.
__device__ __forceinline__ uint32_t near_chunk_bits(uint32_t m) {
  uint32_t b = 8;
  while (m > (kChunkWords * 64) << b) ++b;
  return b;
}

// (grid-stride over the workgroups of the launch)
__device__ __forceinline__ void near_clear(const NearTable& T, uint32_t m, uint32_t start, uint32_t step) {
  const uint32_t slots = pair_table_mask(m) + 1;
  for (uint32_t i = start; i < slots; i += step) {
    T.owner[i] = T.ckey[i] = 0;
#pragma unroll
    for (uint32_t w = 0; w < kChunkWords; ++w) T.bits[(size_t)i * kChunkWords + w] = 0;
  }
}

// Group tables: a slot is 0 or holds its owner (the index that claimed it, plus
// one) and a tag of the owner's hash, so a slot of another key is told apart
// without reading that key. Four slots are read at once. A slot read as empty
// may be stale, which costs the compare-and-swap only; owners never change.
constexpr uint32_t kOwnerBits = 19;
static_assert(kMidMax < 1u << kOwnerBits, "owners fit");
struct Probe {
  uint32_t bucket, pos, tag;  // first slot of the bucket, next slot in it, tag in place
  uint32_t need;              // 1 while the group is not known; then the group is bucket + pos
};
__device__ __forceinline__ Probe probe_start(uint32_t hash, uint32_t mask, bool need) {
  return Probe{hash & mask & ~3u, 0, (hash >> kOwnerBits) << kOwnerBits, need};
}
__device__ __forceinline__ void probe_next(Probe& p, uint32_t mask) {
  if (++p.pos == 4) {
    p.pos = 0;
    p.bucket = (p.bucket + 4) & mask;
  }
}
// Looks through the bucket's words: a word with the key's tag, or 0 with p at
// an empty slot, or kNoSlot with p moved on to the next bucket.
constexpr uint32_t kNoSlot = 0xFFFFFFFFu;
__device__ __forceinline__ uint32_t probe_look(Probe& p, const uint4& v, uint32_t mask) {
  const uint32_t w[4] = {v.x, v.y, v.z, v.w};
  uint32_t hit = 4, o = 0;
#pragma unroll
  for (int k = 3; k >= 0; --k)
    if ((uint32_t)k >= p.pos && (w[k] == 0 || (w[k] >> kOwnerBits) << kOwnerBits == p.tag)) {
      hit = (uint32_t)k;
      o = w[k];
    }
  if (hit == 4) {
    p.bucket = (p.bucket + 4) & mask;
    p.pos = 0;
    return kNoSlot;
  }
  p.pos = hit;
  return o;
}
// The owner + 1 to compare with in the slot's word o, or 0 with p moved on.
__device__ __forceinline__ uint32_t probe_owner(Probe& p, uint32_t o, uint32_t mask) {
  if ((o >> kOwnerBits) << kOwnerBits != p.tag) {  // taken meanwhile, by another key
    probe_next(p, mask);
    return 0;
  }
  return o & ((1u << kOwnerBits) - 1);
}
// One step over the bucket's words: claims the first empty slot for owner own
// (then the group is known: returns 0), or returns the owner + 1 to compare
// with, or 0 with p moved on.
__device__ __forceinline__ uint32_t probe_step(Probe& p, const uint4& v, uint32_t* table, uint32_t mask, uint32_t own) {
  uint32_t o = probe_look(p, v, mask);
  if (o == kNoSlot) return 0;
  if (o == 0) {
    o = atomicCAS(table + p.bucket + p.pos, 0u, p.tag | (own + 1));
    if (o == 0) {
      p.need = 0;
      return 0;
    }
  }
  return probe_owner(p, o, mask);
}
// The same for a whole wavefront (lanes with p.need == 0 take no part), with one
// compare-and-swap for the lanes that want the same empty slot: they agree on
// one of them through the LDS (lead: kLeads words; two slots may meet in one,
// then the lanes of one of the two go alone) and share what it finds. A
// digest that every record carries is wanted by all lanes at once, and swaps of
// one word take 3.4 ns each: 262,144 records of one digest 999 us when every
// lane swapped, 125 us (100,000 records: 351 and 90); logs of fresh digests are
// as fast either way (100,000 records 111 us).
constexpr uint32_t kLeads = 256;
__device__ __forceinline__ uint32_t probe_step_shared(Probe& p, const uint4& v, uint32_t* table, uint32_t mask, uint32_t own,
                                                      uint8_t* lead) {
  const uint32_t lane = threadIdx.x & 63;
  uint32_t o = p.need ? probe_look(p, v, mask) : kNoSlot;
  const uint32_t slot = p.bucket + p.pos;
  if (__ballot(o == 0)) {
    if (o == 0) lead[slot % kLeads] = (uint8_t)lane;
    wave_lds_fence();
    uint32_t by = o == 0 ? lead[slot % kLeads] : lane;
    if ((uint32_t)__shfl((int)slot, (int)by, 64) != slot) by = lane;
    wave_lds_fence();
    uint32_t got = 0;
    if (o == 0 && by == lane) {
      got = atomicCAS(table + slot, 0u, p.tag | (own + 1));
      if (got == 0) {
        p.need = 0;
        got = p.tag | (own + 1);
      }
    }
    got = (uint32_t)__shfl((int)got, (int)by, 64);
    if (o == 0) o = got;
  }
  return p.need && o != kNoSlot ? probe_owner(p, o, mask) : 0u;
}

// Position q's group, by key words a (64 bits) and b (small) of every position.
// All lanes of a wavefront call it and leave it together.
__device__ __forceinline__ uint32_t near_group(const NearTable& T, uint32_t mask, uint32_t q, bool in, const uint64_t* a,
                                               const uint64_t* b) {
  const uint64_t ka = in ? a[q] : 0ull, kb = in ? b[q] : 0ull;
  Probe p = probe_start(near_hash(ka, kb), mask, in);
  while (__ballot(p.need)) {
    if (!p.need) continue;
    const uint32_t o = probe_step(p, *reinterpret_cast<const uint4*>(T.owner + p.bucket), T.owner, mask, q);
    if (o) {
      if (a[o - 1] == ka && b[o - 1] == kb) p.need = 0; else probe_next(p, mask);
    }
  }
  return p.bucket + p.pos;
}

__device__ __forceinline__ uint32_t near_slot(const NearTable& T, uint32_t mask, uint32_t g, uint32_t chunk, bool insert) {
  const uint32_t key = (g << 8 | chunk) + 1;
  uint32_t h = near_hash(key, 0) & mask;
  for (;;) {
    uint32_t o = T.ckey[h];
    if (o == 0 && insert) o = atomicCAS(T.ckey + h, 0u, key);
    if (o == 0 || o == key) break;
    h = (h + 1) & mask;
  }
  return h;
}

struct NearLds {
  uint64_t a[kChunkMax];
  alignas(8) uint16_t slot[kChunkMax];  // per position: its key's slot below, kNoGroup16 past the list
  uint32_t owner[2 * kChunkMax];    // a position of the key; then the key's group
  uint32_t rounds[2 * kChunkMax];   // which stretches of 64 positions hold the key
  uint8_t b[kChunkMax];
};
constexpr uint32_t kNoGroup16 = 0xFFFF;
static_assert(kChunkMax <= 32 * 64, "a bit per stretch of 64");

// Enters the chunks first, first + step, ... of the list, by a workgroup of kT
// threads: keys a (64 bits) and b (below 256) of every position. In LDS an exact
// hash table of the chunk's keys; ballots over its slot numbers give the
// neighbours inside 64 positions, a bit per stretch of 64 the others. Bound by
// the latency of its LDS and table accesses.
template <bool REV>
__device__ void near_enter(const NearTable& T, uint32_t m, const uint64_t* a, const uint64_t* b, NearLds& L, uint32_t first,
                           uint32_t step) {
  constexpr uint32_t kFree = 0xFFFFFFFFu, kSlots = 2 * kChunkMax;
  constexpr int kR = kChunkMax / kT;
  const uint32_t mask = pair_table_mask(m), cb = near_chunk_bits(m), size = 1u << cb;
  const uint32_t t = threadIdx.x, lane = t & 63;
  const uint64_t lt = lanemask_lt();
  uint16_t* const slot = L.slot;
  for (uint32_t c = first; (uint64_t)c << cb < m; c += step) {
    const uint32_t base = c << cb;
    __syncthreads();
    for (uint32_t x = t; x < kSlots; x += kT) {
      L.owner[x] = kFree;
      L.rounds[x] = 0;
    }
    uint64_t ka[kR], kb[kR];
#pragma unroll
    for (int r = 0; r < kR; ++r) {
      const uint32_t i = r * kT + t, p = base + i;
      ka[r] = kb[r] = 0;
      if (i < size && p < m) {
        ka[r] = a[REV ? m - 1 - p : p];
        kb[r] = b[REV ? m - 1 - p : p];
      }
    }
#pragma unroll
    for (int r = 0; r < kR; ++r) {
      L.a[r * kT + t] = ka[r];
      L.b[r * kT + t] = (uint8_t)kb[r];
    }
    __syncthreads();
    for (uint32_t i = t; i < size; i += kT) {
      uint32_t s = kNoGroup16;
      if (base + i < m) {
        const uint64_t x = L.a[i];
        const uint8_t y = L.b[i];
        s = (near_hash(x, y) >> 8) % kSlots;
        for (;;) {
          uint32_t o = L.owner[s];
          if (o == kFree) o = atomicCAS(&L.owner[s], kFree, i);
          if (o == kFree || (L.a[o] == x && L.b[o] == y)) break;
          s = (s + 1) % kSlots;
        }
      }
      slot[i] = (uint16_t)s;
    }
    __syncthreads();
    // bit r: of this thread's position r * kT + t, whether it owns its slot and
    // whether it is the key's first or last in its 64 positions
    uint32_t owns = 0, firsts = 0, lasts = 0;
    for (uint32_t i = t, r = 0; i < size; i += kT, ++r) {
      const uint32_t s = slot[i], in = s != kNoGroup16;
      uint64_t peers = __ballot(in);
#pragma unroll
      for (int k = 0; k < 11; ++k) {
        const bool bit = (s >> k) & 1;
        const uint64_t x = __ballot(bit);
        peers &= bit ? x : ~x;
      }
      if (!in) continue;
      if (peers & lt) {
        T.link[base + i] = base + i - lane + 63 - (uint32_t)__builtin_clzll(peers & lt);
      } else {
        firsts |= 1u << r;
        atomicOr(&L.rounds[s], 1u << (i >> 6));
      }
      if ((peers & ~lt) == 1ull << lane) lasts |= 1u << r;
      if (L.owner[s] == i) owns |= 1u << r;
    }
    __syncthreads();
    for (uint32_t i = t, r = 0; i < size; i += kT, ++r) {
      const bool own = (owns >> r) & 1;
      const uint32_t p = base + i, g = near_group(T, mask, REV ? m - 1 - p : p, own, a, b);
      if (own) L.owner[slot[i]] = g;
    }
    __syncthreads();
    for (uint32_t i = t, r = 0; i < size; i += kT, ++r) {
      if (!(((firsts | lasts) >> r) & 1)) continue;
      const uint32_t s = slot[i], x = i >> 6, rounds = L.rounds[s], g = L.owner[s];
      if ((firsts >> r) & 1) {
        const uint32_t earlier = rounds & ((1u << x) - 1);
        uint32_t v = kFar | g;
        if (earlier) {  // the last of them in that stretch, four at a time
          const uint32_t y = 31 - (uint32_t)__builtin_clz(earlier);
          uint32_t found = kFree;
          for (uint32_t u = y * 16 + 16; found == kFree;) {
            uint64_t four;
            __builtin_memcpy(&four, slot + 4 * --u, 8);
#pragma unroll
            for (uint32_t k = 0; k < 4; ++k)
              if (((four >> (16 * k)) & 0xFFFF) == s) found = u * 4 + k;
          }
          v = base + found;
        }
        T.link[base + i] = v;
      }
      if (((lasts >> r) & 1) && rounds >> x == 1) {  // its last in the chunk
        T.clast[near_slot(T, mask, g, c, true)] = base + i;
        atomicOr(T.bits + (size_t)g * kChunkWords + (c >> 6), 1ull << (c & 63));
      }
    }
  }
}

// The nearest earlier position of p's group, or kNone. (A launch after near_enter's.)
__device__ __forceinline__ uint32_t near_prev(const NearTable& T, uint32_t m, uint32_t p) {
  const uint32_t v = T.link[p];
  if (!(v & kFar)) return v;
  const uint32_t g = v & ~kFar, c = p >> near_chunk_bits(m);
  for (int w = (int)(c >> 6); w >= 0; --w) {
    unsigned long long x = T.bits[(size_t)g * kChunkWords + w];
    if (w == (int)(c >> 6)) x &= (1ull << (c & 63)) - 1;
    if (x) return T.clast[near_slot(T, pair_table_mask(m), g, (uint32_t)w * 64 + 63 - (uint32_t)__builtin_clzll(x), false)];
  }
  return kNone;
}

struct MidView {
  uint32_t *gid0, *gid1;   // digest group of each record (kNone: no transfer); of each element after the first pass
  uint32_t* dtab;          // digest table: 1 + the record that claimed the slot
  uint32_t *h0, *h1;       // [tiles][digits] of the two passes
  uint8_t* uth;            // per record: 1 for an unused transfer
  uint64_t *ad_host, *ad_bytes;  // per ALLOC/DELETE: host address, bytes
  uint64_t* kd_te;         // per kernel of the per-device lists: end
  uint64_t *ks, *ke;       // starts and ends of the lists, each sorted by tiles of kKernTile (not chronological logs)
  NearTable ad, ut;
  WaveScan wscan;
  WaveAgg* agg;
  Parts parts;
};

// ---------------------------------------------------------------------------
// Digest path.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kMidT) void mid_clear_kernel(uint32_t* dtab, uint32_t slots, uint32_t* hist, uint32_t nhist,
                                                          AnaCtl* ctl, uint32_t n) {
  const uint32_t t = blockIdx.x * kMidT + threadIdx.x;
  for (uint32_t i = t; i < slots; i += gridDim.x * kMidT) dtab[i] = 0;
  for (uint32_t i = t; i < nhist; i += gridDim.x * kMidT) hist[i] = 0;
  if (blockIdx.x == 0 && threadIdx.x < kScanQ) ctl->scan_tq[threadIdx.x] = 0;
  if (t == 0) {
    ctl->n = n;
    ctl->ut_need_sort = ctl->scan_ticket = 0;
  }
}

struct MidClassify {
  const odp_event* ev;
  uint32_t n;
  uint8_t *flags, *cls, *uth;
  uint32_t *gid, *val;
  uint32_t* wave_cnt;
  uint64_t* wave_kmax;
  uint32_t *dtab, dmask;
  uint32_t* hist;
  uint32_t bits;
  Parts parts;
};

// 256 threads and one record each: a workgroup's time is a chain of memory
// round trips (record, table, compare-and-swap), so the log is spread over as
// many compute units as there are (100,000 records: 30 us with workgroups of
// 2,048 records, 18 us with 256). The first pass's tile histograms are summed by
// atomics then (kMidTile / 256 workgroups each).
constexpr int kClsT = 256, kClsRounds = 1;
constexpr uint32_t kClsWave = 64 * kClsRounds;
__global__ __launch_bounds__(kClsT) void mid_classify_kernel(MidClassify A) {
  constexpr int kW = kClsT / 64, R = kClsRounds;
  __shared__ uint32_t s_kdev[kW][kEp];
  __shared__ unsigned long long s_kmax[kW][kEp];
  __shared__ uint32_t s_h[kMidDigits];
  __shared__ uint8_t s_lead[kW][kLeads];
  const odp_event* __restrict__ ev = A.ev;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const uint32_t n = A.n, wid = blockIdx.x * kW + w, wb = wid * kClsWave;
  for (uint32_t d = threadIdx.x; d < (1u << A.bits); d += kClsT) s_h[d] = 0;
  if (lane < kEp) {
    s_kdev[w][lane] = 0;
    s_kmax[w][lane] = 0;
  }
  __syncthreads();
  odp_event e[R];
  uint64_t before[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const uint32_t i = wb + r * 64 + lane;
    before[r] = 0;
    if (i < n) {
      e[r] = ev[i];
      if (i) before[r] = ev[i - 1].t_start;
    }
  }
  unsigned long long n_inv = 0, n_tx = 0, n_k = 0, tmin = ~0ull, tmax = 0;
  uint32_t bad = kNone, mep = 0, c_ad = 0, c_k = 0, c_ut = 0;
  uint32_t code[R];
  Probe pr[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const uint32_t i = wb + r * 64 + lane;
    uint8_t c = C_INVALID;
    code[r] = kNotTransfer;
    pr[r] = Probe{0, 0, 0, 0};
    if (i < n) {
      const odp_event& x = e[r];
      const bool is_tx = x.op == ODP_H2D || x.op == ODP_D2H || x.op == ODP_D2D;
      const bool valid = x.op >= ODP_ALLOC && x.op <= ODP_KERNEL && x.t_end >= x.t_start && x.t_start >= before[r] &&
                         dev_ok(x.dst_dev) && (!is_tx || dev_ok(x.src_dev));
      if (valid) {
        tmin = min(tmin, (unsigned long long)x.t_start);
        tmax = max(tmax, (unsigned long long)x.t_end);
        if (is_tx) {
          c = x.op != ODP_D2H && x.dst_dev >= 0 ? C_COPYIN : C_TRANSFER;
          code[r] = pack_ep((uint32_t)(x.src_dev + 1), (uint32_t)(x.dst_dev + 1));
          mep = max(mep, (uint32_t)max(x.src_dev + 1, x.dst_dev + 1));
          pr[r] = probe_start(near_hash(x.digest, 0), A.dmask, true);
          ++n_tx;
        } else if (x.op == ODP_KERNEL) {
          c = C_KERNEL;
          ++n_k;
          atomicAdd(&s_kdev[w][x.dst_dev + 1], 1u);
          atomicMax(&s_kmax[w][x.dst_dev + 1], (unsigned long long)x.t_end);
        } else {
          c = C_ALLOCDEL;
        }
      } else {
        ++n_inv;
        bad = min(bad, i);
      }
      A.flags[i] = valid ? 0 : ODP_F_INVALID;
      A.cls[i] = c;
      A.uth[i] = 0;
    }
    c_ad += (uint32_t)__popcll(__ballot(c == C_ALLOCDEL));
    c_k += (uint32_t)__popcll(__ballot(c == C_KERNEL));
    c_ut += (uint32_t)__popcll(__ballot(c == C_COPYIN));
  }
  // Digest groups: all rounds' probes in flight together. The loop runs while
  // any lane of the wavefront probes, so all lanes leave it together.
  for (;;) {
    uint32_t any = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) any |= pr[r].need;
    if (!__ballot(any)) break;
    uint4 v[R];
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (pr[r].need) v[r] = *reinterpret_cast<const uint4*>(A.dtab + pr[r].bucket);
    uint32_t o[R];
#pragma unroll
    for (int r = 0; r < R; ++r) o[r] = probe_step_shared(pr[r], v[r], A.dtab, A.dmask, wb + r * 64 + lane, s_lead[w]);
    uint64_t od[R];
#pragma unroll
    for (int r = 0; r < R; ++r) od[r] = o[r] ? ev[o[r] - 1].digest : 0ull;
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (o[r]) {
        if (od[r] == e[r].digest) pr[r].need = 0; else probe_next(pr[r], A.dmask);
      }
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const uint32_t i = wb + r * 64 + lane;
    if (i < n) {
      const bool tx = code[r] != kNotTransfer;
      const uint32_t g = pr[r].bucket + pr[r].pos;
      A.gid[i] = tx ? g : kNone;
      A.val[i] = i | code[r] << 24;
      if (tx) atomicAdd(&s_h[g & ((1u << A.bits) - 1)], 1u);
    }
  }
  if (lane == 0) {
    A.wave_cnt[kWaveCnt * wid] = c_ad;
    A.wave_cnt[kWaveCnt * wid + 1] = c_k;
    A.wave_cnt[kWaveCnt * wid + 2] = c_ut;
  }
  __syncthreads();
  const uint32_t tile = blockIdx.x / (kMidTile / (kClsT * kClsRounds));
  for (uint32_t d = threadIdx.x; d < (1u << A.bits); d += kClsT)
    if (s_h[d]) atomicAdd(A.hist + ((size_t)tile << A.bits | d), s_h[d]);
  if (lane < kEp) {
    A.wave_cnt[kWaveCnt * wid + 3 + lane] = s_kdev[w][lane];
    A.wave_kmax[kEp * wid + lane] = s_kmax[w][lane];
  }
  block_store<R_ADD, kClsT>(A.parts.at(S_N_INVALID), n_inv);
  block_store<R_ADD, kClsT>(A.parts.at(S_N_TRANSFERS), n_tx);
  block_store<R_ADD, kClsT>(A.parts.at(S_N_KERNELS), n_k);
  block_store<R_MIN, kClsT>(A.parts.at(S_FIRST_BAD), bad);
  block_store<R_MAX, kClsT>(A.parts.at(S_MAX_EP), mep);
  block_store<R_MIN, kClsT>(A.parts.at(S_TMIN), tmin);
  block_store<R_MAX, kClsT>(A.parts.at(S_TMAX), tmax);
}

// The wavefront scans and, in further workgroups, the classification's sums.
constexpr uint32_t kMidSums = 7;
__global__ __launch_bounds__(kMidT) void mid_scan_kernel(WaveScan S, uint32_t nchunk, AnaCtl* ctl, Parts parts, uint32_t nb,
                                                         odp_report* rep, SortJob* big) {
  if (blockIdx.x < nchunk * kScanQ) {
    wave_scan_body(S, nchunk, ctl);
    return;
  }
  constexpr uint32_t kSlot[kMidSums] = {S_N_INVALID, S_N_TRANSFERS, S_N_KERNELS, S_FIRST_BAD, S_MAX_EP, S_TMIN, S_TMAX};
  const uint32_t k = blockIdx.x - nchunk * kScanQ;
  reduce_slot<kMidT>(parts, nb, kSlot[k], ctl, rep);
  if (k == 0 && threadIdx.x == 0) {
    big->npasses = 2;  // the sorted order ends in keys[0], vals[0], and holds every transfer
    big->n_after1 = nullptr;
  }
}

// One pass of the stable sort by group number: a tile of kMidTile elements per
// workgroup. Digit d of all tiles is summed by thread d, which gives the
// global start of the digit and of this tile's share of it without a scan
// launch between (128 tiles at most).
constexpr uint32_t kMidCols = 32;
__global__ __launch_bounds__(kMidT) void mid_scatter_kernel(uint32_t pass, uint32_t n, const AnaCtl* ctl, uint32_t bits,
                                                            const uint32_t* __restrict__ hist,
                                                            const uint32_t* __restrict__ gid,
                                                            const uint32_t* __restrict__ val, uint32_t* gid_out,
                                                            unsigned long long* key_out, uint32_t* val_out) {
  constexpr int kW = kMidT / 64, R = kMidRounds;
  __shared__ uint32_t s_cnt[kW * kMidDigits];
  __shared__ uint32_t s_wt[16];
  const uint32_t nel = pass == 0 ? n : ctl->n_tx, tb = blockIdx.x * kMidTile;
  if (tb >= nel) return;
  const uint32_t t = threadIdx.x, lane = t & 63, w = t >> 6, nd = 1u << bits, shift = pass * bits;
  const uint32_t tiles = (nel + kMidTile - 1) / kMidTile;
  uint32_t g[R], v[R], rk[R], dg[R], in[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const uint32_t j = tb + w * kMidWave + r * 64 + lane;
    g[r] = j < nel ? gid[j] : kNone;
    v[r] = j < nel ? val[j] : 0u;
    in[r] = g[r] != kNone;
    dg[r] = in[r] ? (g[r] >> shift) & (nd - 1) : 0u;
  }
  uint32_t earlier = 0, all = 0;
  if (t < nd) {
    // (kMidCols tiles' counts in flight together: with 8, and the last ones one
    // by one, these reads took most of the kernel: 200,000 records 24 -> 17 us)
    for (uint32_t x0 = 0; x0 < tiles; x0 += kMidCols) {
      uint32_t c[kMidCols];
#pragma unroll
      for (uint32_t u = 0; u < kMidCols; ++u) c[u] = hist[(size_t)min(x0 + u, tiles - 1) << bits | t];
#pragma unroll
      for (uint32_t u = 0; u < kMidCols; ++u) {
        const uint32_t x = x0 + u;
        earlier += x < blockIdx.x ? c[u] : 0u;
        all += x < tiles ? c[u] : 0u;
      }
    }
  }
  for (uint32_t x = t; x < kW * nd; x += kMidT) s_cnt[x] = 0;
  __syncthreads();
  uint32_t* const mine = s_cnt + w * nd;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    uint64_t peers = __ballot(in[r]);
    for (uint32_t b = 0; b < bits; ++b) {
      const bool bit = (dg[r] >> b) & 1;
      const uint64_t m = __ballot(bit);
      peers &= bit ? m : ~m;
    }
    const uint32_t before = in[r] ? mine[dg[r]] : 0u;
    rk[r] = before + (uint32_t)__popcll(peers & lanemask_lt());
    wave_lds_fence();
    if (in[r] && (peers >> lane) == 1ull) mine[dg[r]] = before + (uint32_t)__popcll(peers);
    wave_lds_fence();
  }
  uint32_t total;
  const uint32_t start = block_xscan<uint32_t, false>(all, s_wt, total);  // (its barriers order s_cnt too)
  if (t < nd) {
    uint32_t run = start + earlier;
    for (int x = 0; x < kW; ++x) {
      const uint32_t c = s_cnt[x * nd + t];
      s_cnt[x * nd + t] = run;
      run += c;
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if (!in[r]) continue;
    const uint32_t p = mine[dg[r]] + rk[r];
    if (pass == 0) gid_out[p] = g[r]; else key_out[p] = g[r];
    val_out[p] = v[r];
  }
}

__global__ __launch_bounds__(kMidT) void mid_hist_kernel(const AnaCtl* ctl, uint32_t bits, const uint32_t* __restrict__ gid,
                                                         uint32_t* __restrict__ hist) {
  __shared__ uint32_t s_h[kMidDigits];
  const uint32_t nel = ctl->n_tx, tb = blockIdx.x * kMidTile, t = threadIdx.x, nd = 1u << bits;
  if (tb >= nel) return;
  s_h[t] = 0;
  uint32_t g[kMidRounds];
#pragma unroll
  for (int r = 0; r < kMidRounds; ++r) {
    const uint32_t j = tb + r * kMidT + t;
    g[r] = j < nel ? gid[j] : kNone;
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kMidRounds; ++r)
    if (g[r] != kNone) atomicAdd(&s_h[(g[r] >> bits) & (nd - 1)], 1u);
  __syncthreads();
  if (t < nd) hist[(size_t)blockIdx.x << bits | t] = s_h[t];
}

// ---------------------------------------------------------------------------
// Allocation and unused-transfer path.
// ---------------------------------------------------------------------------
struct MidSide {
  const odp_event* ev;
  const uint8_t* cls;
  uint32_t n;
  WaveScan W;
  SubsetOut S;
  MidView M;
  PairTable T;
  UtArgs U;
  uint8_t* flags;
  AnaCtl* ctl;
};

// Ordered compaction of the subsets (as subset_scatter_kernel, a round per
// wavefront), and the clearing of the tables that the next launches fill.
__global__ __launch_bounds__(kT) void mid_subset_kernel(MidSide A) {
  const AnaCtl* c = A.ctl;
  {
    const uint32_t start = blockIdx.x * kT + threadIdx.x, step = gridDim.x * kT;
    near_clear(A.M.ad, c->n_ad, start, step);
    near_clear(A.M.ut, c->n_ut, start, step);
    const uint32_t slots = pair_table_mask(c->n_ad / 2) + 1;
    for (uint32_t i = start; i < slots; i += step) {
      A.T.owner[i] = 0;
      A.T.first[i] = kNone;
      A.T.multi[i] = 0;
    }
  }
  subset_scatter_body<kClsRounds, true>(A.ev, A.cls, A.n, A.W, A.S, Parts{}, A.M.ad_host, A.M.ad_bytes, A.M.kd_te);
}

// Unused transfers by the forward search, and the groups of the ALLOC/DELETE
// records.
// The forward search goes over a longer stretch here: a log whose devices each
// run a kernel every few hundred copies needs no group table for its copies then (with 64 copies ahead, 200,000 records on three devices did: the
// table's insertion and lookups took 340 us).
constexpr uint32_t kMidWindow = 1024;
constexpr uint32_t kMidStage = kT + kMidWindow;
struct UtLds {
  uint32_t ix[kMidStage], h[kMidStage + 8];  // (read eight at a time)
};
constexpr uint32_t kKernTile = 2048;
union LinkLds {
  UtLds ut;
  NearLds near;
  uint64_t kern[kKernTile];
};
__device__ void mid_ut_scan(const MidSide& A, UtLds& L, uint32_t block, uint32_t nblocks) {
  const UtArgs& U = A.U;
  const uint32_t n = *U.n_ut;
  if (U.ctl->first_bad != kNone) {
    if (n && block == 0 && threadIdx.x == 0) U.ctl->ut_need_sort = 1;
    return;
  }
  uint32_t *const s_ix = L.ix, *const s_h = L.h;
  for (uint32_t b0 = block * kT; b0 < n; b0 += nblocks * kT) {
    // s_*[x] holds copy-in b0 + 1 + x (index kNone past the last)
    for (uint32_t x = threadIdx.x; x < kMidStage; x += kT) {
      const uint32_t r = b0 + 1 + x;
      s_ix[x] = r < n ? U.ut_idx[r] : kNone;
      s_h[x] = r < n ? A.S.ut_vals[r] : 0u;
    }
    __syncthreads();
    const uint32_t q = b0 + threadIdx.x;
    if (q < n) {
      const uint8_t hit = ut_decide<kMidWindow, kMidWindow>(U, s_ix, s_h, b0, q, A.S.ut_vals[q]);
      U.ut_hit[q] = hit;
      if (hit == 1) A.M.uth[U.ut_idx[q]] = 1;
      if (hit == 2) U.ctl->ut_need_sort = 1;
    }
    __syncthreads();
  }
}

// In a log that is not chronological: the starts and the ends of each device's
// kernels, sorted in tiles of kKernTile (a workgroup each, in LDS), for the count
// form's binary searches (mid_kernels_meeting).
__device__ void mid_sort_kernels(const MidSide& A, uint64_t* s, uint32_t block, uint32_t nblocks) {
  uint32_t job = block;  // (device, tile, starts or ends)
  for (int d = 0; d < kEp; ++d) {
    const uint32_t total = A.ctl->kd_total[d], jobs = 2 * ((total + kKernTile - 1) / kKernTile);
    for (; job < jobs; job += nblocks) {
      const uint32_t at = job / 2 * kKernTile, len = min(kKernTile, total - at);
      const uint64_t* from = (job & 1 ? A.M.kd_te : A.S.kd_ts) + A.ctl->kd_base[d] + at;
      uint64_t* to = (job & 1 ? A.M.ke : A.M.ks) + A.ctl->kd_base[d] + at;
      uint32_t top = 2;
      while (top < len) top <<= 1;
      __syncthreads();
      for (uint32_t x = threadIdx.x; x < top; x += kT) s[x] = x < len ? from[x] : ~0ull;
      __syncthreads();
      for (uint32_t k = 2; k <= top; k <<= 1)  // bitonic
        for (uint32_t j = k >> 1; j > 0; j >>= 1) {
          for (uint32_t x = threadIdx.x; x < top / 2; x += kT) {
            const uint32_t i = (x & ~(j - 1)) << 1 | (x & (j - 1)), o = i | j;
            const uint64_t a = s[i], b = s[o];
            if ((a > b) == ((i & k) == 0)) {
              s[i] = b;
              s[o] = a;
            }
          }
          __syncthreads();
        }
      for (uint32_t x = threadIdx.x; x < len; x += kT) to[x] = s[x];
    }
    job -= jobs;
  }
}

// Half of the workgroups each: both are chains of memory round trips.
__global__ __launch_bounds__(kT) void mid_link_kernel(MidSide A) {
  __shared__ LinkLds L;
  const uint32_t half = gridDim.x / 2;
  if (blockIdx.x >= half) {
    mid_ut_scan(A, L.ut, blockIdx.x - half, half);
    if (A.ctl->first_bad != kNone) mid_sort_kernels(A, L.kern, blockIdx.x - half, half);
    return;
  }
  near_enter<false>(A.M.ad, A.ctl->n_ad, A.S.ad_w_addr, A.S.ad_w_dev, L.near, blockIdx.x, half);
}

// Enters the wavefront's paired ALLOCs (positions k of the lanes with in) in the
// RA table. Lanes of one key agree on one of them (as probe_step_shared; two
// keys that meet in a lead word: one of the two goes lane by lane), which
// enters the smallest position for all: a program that maps one array again and
// again would send every swap and minimum to the same words (131,072 pairs of
// one array: the whole analysis 310 us, and 106 so).
struct RaLds {
  uint32_t least[64];  // per leading lane: the smallest position of its lanes
  uint8_t several[64], lead[kLeads];
};
__device__ __forceinline__ void mid_ra_insert(const MidSide& A, uint32_t tmask, uint32_t k, bool in, RaLds& L) {
  if (!__ballot(in)) return;
  const uint32_t lane = threadIdx.x & 63;
  const uint64_t ha = in ? A.M.ad_host[k] : 0, dv = in ? A.S.ad_w_dev[k] : 0, by = in ? A.M.ad_bytes[k] : 0;
  const uint32_t h = pair_hash(ha, dv, by);
  L.least[lane] = kNone;
  L.several[lane] = 0;
  if (in) L.lead[h % kLeads] = (uint8_t)lane;
  wave_lds_fence();
  uint32_t l = in ? L.lead[h % kLeads] : lane;
  const bool same = __shfl(ha, (int)l, 64) == ha && __shfl(dv, (int)l, 64) == dv && __shfl(by, (int)l, 64) == by;
  if (!same) l = lane;
  if (in) atomicMin(&L.least[l], k);
  if (in && l != lane) L.several[l] = 1;
  wave_lds_fence();
  uint32_t t = h & tmask;
  if (in && l == lane) {
    // what the probe loop's lanes decide is stored inside it: they leave it at different trips
    for (;; t = (t + 1) & tmask) {
      uint32_t o = A.T.owner[t];
      if (o == 0) o = atomicCAS(A.T.owner + t, 0u, k + 1);
      if (o == 0) {  // claimed
        if (L.several[lane]) A.T.multi[t] = 1;
        break;
      }
      if (same_pair_key(A.M.ad_host, A.S.ad_w_dev, A.M.ad_bytes, o - 1, k)) {  // joined
        if (A.T.multi[t] == 0) A.T.multi[t] = 1;
        break;
      }
    }
    if (L.least[lane] < A.T.first[t]) atomicMin(A.T.first + t, L.least[lane]);
  }
  t = (uint32_t)__shfl((int)t, (int)l, 64);
  if (in) A.T.slot[k] = t;
  wave_lds_fence();
}

// Pairing (a DELETE with its predecessor of the same device address, when that
// is an ALLOC) and the RA table; when the forward search left copies open, the
// groups of the copies' places.
__global__ __launch_bounds__(kT) void mid_pair_kernel(MidSide A) {
  const AnaCtl* c = A.ctl;
  const uint32_t m = c->n_ad, tmask = pair_table_mask(m / 2);
  const uint32_t lane = threadIdx.x & 63;
  __shared__ RaLds s_ra[kT / 64];
  for (uint32_t b = (blockIdx.x * kT + threadIdx.x) / 64 * 64; b < m; b += gridDim.x * kT) {
    const uint32_t q = b + lane;
    const bool del = q < m && A.S.ad_op[q] == ODP_DELETE;
    const uint32_t p = del ? near_prev(A.M.ad, m, q) : kNone;
    const bool paired = p != kNone && A.S.ad_op[p] == ODP_ALLOC;
    if (paired) {
      A.S.ad_alloc_partner[p] = q;
      A.flags[A.S.ad_idx[q]] = ODP_F_PAIRED;
    }
    mid_ra_insert(A, tmask, p, paired, s_ra[threadIdx.x >> 6]);
  }
  if (c->ut_need_sort) {
    __shared__ NearLds L;
    near_enter<true>(A.M.ut, c->n_ut, A.S.ut_w_addr, A.S.ut_w_code, L, blockIdx.x, gridDim.x);
  }
}

// Kernels of device code dev that start by hi, less those that end before lo
// (modulo 2^32): the count form, in any kernel order, tile by tile. A tile on one
// side of a bound, as most are where only a stretch of the log is out of
// order, needs no search. (By extremes of 64 and 4,096 kernels in log order
// instead of sorted tiles, each query went through hundreds of them: 200,000
// records, 3 of them rejected, 760 us; 192 us so.)
__device__ __forceinline__ uint32_t mid_kernels_meeting(const MidSide& A, uint32_t dev, uint64_t lo, uint64_t hi) {
  const uint32_t total = A.ctl->kd_total[dev], base = A.ctl->kd_base[dev];
  uint32_t cnt = 0;
  for (uint32_t at = 0; at < total; at += kKernTile) {
    const uint32_t len = min(kKernTile, total - at);
    const uint64_t *ks = A.M.ks + base + at, *ke = A.M.ke + base + at;
    const uint64_t s0 = ks[0], s1 = ks[len - 1], e0 = ke[0], e1 = ke[len - 1];
    uint32_t started = s0 > hi ? 0u : len, ended = e0 >= lo ? 0u : len;
    if ((started && s1 > hi) || (ended && e1 >= lo)) {
      // both searches take the same steps, so their loads are in flight together
      uint32_t a = 0, b = 0, left = len;
      for (; left > 1; left -= left / 2) {
        const uint32_t half = left / 2;
        const uint64_t x = ks[a + half - 1], y = ke[b + half - 1];
        a += x <= hi ? half : 0u;
        b += y < lo ? half : 0u;
      }
      started = a + (ks[a] <= hi);
      ended = b + (ke[b] < lo);
    }
    cnt += started - ended;
  }
  return cnt;
}

// Flags and sums of the ALLOC/DELETE records, and the copies that the forward
// search left open.
__global__ __launch_bounds__(kT) void mid_ra_ua_kernel(MidSide A) {
  const AnaCtl* ctl = A.ctl;
  const odp_event* __restrict__ ev = A.ev;
  const bool chrono = ctl->first_bad == kNone;
  const uint32_t m = ctl->n_ad;
  unsigned long long c_pair = 0, c_unp = 0, c_ra = 0, c_grp = 0, b_ra = 0, t_ra = 0, c_ua = 0, b_ua = 0, t_ua = 0, t_el = 0;
  for (uint32_t q = blockIdx.x * kT + threadIdx.x; q < m; q += gridDim.x * kT) {
    if (A.S.ad_op[q] != ODP_ALLOC) continue;
    const uint32_t p = A.S.ad_alloc_partner[q];
    if (p == kNone) {
      ++c_unp;
      continue;
    }
    ++c_pair;
    const uint32_t t = A.T.slot[q], ai = A.S.ad_idx[q];
    const odp_event &a = ev[ai], &d = ev[A.S.ad_idx[p]];
    const uint64_t dur = (a.t_end - a.t_start) + (d.t_end - d.t_start);
    const bool head = A.T.first[t] == q;
    uint8_t f = ODP_F_PAIRED;
    if (!head) {
      f |= ODP_F_RA;
      ++c_ra;
      b_ra += a.bytes;
      t_ra += dur;
    }
    c_grp += head && A.T.multi[t] != 0;
    const uint32_t dev = (uint32_t)A.S.ad_w_dev[q];
    bool used;
    if (chrono) {
      const uint32_t ka = A.S.ad_kc[q], kd = A.S.ad_kc[p];
      used = (ka > 0 && A.S.ad_km[q] >= a.t_start) || kd != ka ||
             (kd < ctl->kd_total[dev] && A.S.kd_ts[ctl->kd_base[dev] + kd] <= d.t_end);
    } else {
      used = mid_kernels_meeting(A, dev, a.t_start, d.t_end) != 0;
    }
    if (!used) {
      f |= ODP_F_UA;
      ++c_ua;
      b_ua += a.bytes;
      t_ua += dur;
    }
    if (f & (ODP_F_RA | ODP_F_UA)) t_el += dur;
    A.flags[ai] = f;
  }
  if (ctl->ut_need_sort) {
    const uint32_t n = ctl->n_ut;
    for (uint32_t q = blockIdx.x * kT + threadIdx.x; q < n; q += gridDim.x * kT) {
      if (chrono && A.U.ut_hit[q] != 2) continue;
      const uint32_t dev = (uint32_t)(A.S.ut_w_code[q] & 15), np = near_prev(A.M.ut, n, n - 1 - q);
      const uint32_t nq = np == kNone ? kNone : n - 1 - np;  // (the list was entered backwards)
      const uint64_t ts = A.S.ut_ts[q];
      bool read;
      if (chrono) {
        const uint32_t k = A.S.ut_kc[q], cnt = ctl->kd_total[dev];
        read = k > 0 && A.S.ut_km[q] >= ts;
        if (!read && nq != kNone) {
          const uint32_t kn = A.S.ut_kc[nq];
          read = kn != k || (kn < cnt && A.S.kd_ts[ctl->kd_base[dev] + kn] == A.S.ut_ts[nq]);
        } else if (!read) {
          read = k != cnt;
        }
      } else {
        read = mid_kernels_meeting(A, dev, ts, nq != kNone ? A.S.ut_ts[nq] : ~0ull) != 0;
      }
      if (!read) A.M.uth[A.S.ut_idx[q]] = 1;
    }
  }
  block_store<R_ADD>(A.M.parts.at(S_PAIRS), c_pair);
  block_store<R_ADD>(A.M.parts.at(S_UNP_ALLOC), c_unp);
  block_store<R_ADD>(A.M.parts.at(S_RA_EVENTS), c_ra);
  block_store<R_ADD>(A.M.parts.at(S_RA_GROUPS), c_grp);
  block_store<R_ADD>(A.M.parts.at(S_RA_BYTES), b_ra);
  block_store<R_ADD>(A.M.parts.at(S_RA_TIME), t_ra);
  block_store<R_ADD>(A.M.parts.at(S_UA_EVENTS), c_ua);
  block_store<R_ADD>(A.M.parts.at(S_UA_BYTES), b_ua);
  block_store<R_ADD>(A.M.parts.at(S_UA_TIME), t_ua);
  block_store<R_ADD>(A.M.parts.at(S_ELIM_PAIRS), t_el);
}

// ---------------------------------------------------------------------------
// All sums into the report, by one workgroup: nd partials of the digest path's
// last launch, na of the allocation path's.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kMidT) void mid_finish_kernel(Parts parts, uint32_t nd, uint32_t na, uint32_t n, AnaCtl* ctl,
                                                           odp_report* rep) {
  __shared__ unsigned long long s_sum[kSlots];
  const uint32_t lane = threadIdx.x & 63;
  for (uint32_t k = S_DD_EVENTS + (threadIdx.x >> 6); k < kSlots; k += kMidT / 64) {
    const bool digest = k <= S_ELIM_TX || (k >= S_UT_EVENTS && k <= S_UT_TIME);
    const uint32_t nb = k == S_ELIM_UT ? 0u : digest ? nd : na;  // (the digest path counts a transfer's time once)
    unsigned long long v = 0;
    for (uint32_t b = lane; b < nb; b += 64) v += parts.p[(size_t)k * parts.stride + b];
    v = wave_sum(v);
    if (lane == 0) s_sum[k] = v;
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  const unsigned long long* s = s_sum;
  rep->n_events = n;
  rep->n_alloc_pairs = s[S_PAIRS];
  rep->n_unpaired_alloc = s[S_UNP_ALLOC];
  rep->n_unpaired_delete = ctl->n_ad - s[S_UNP_ALLOC] - 2 * s[S_PAIRS];
  rep->dd_events = s[S_DD_EVENTS];
  rep->dd_groups = s[S_DD_GROUPS];
  rep->dd_members = s[S_DD_EVENTS] + s[S_DD_GROUPS];
  rep->dd_bytes = s[S_DD_BYTES];
  rep->dd_time_ns = s[S_DD_TIME];
  rep->rt_pairs = s[S_RT_PAIRS];
  rep->rt_rx_events = s[S_RT_RX];
  rep->rt_bytes = s[S_RT_BYTES];
  rep->rt_time_ns = s[S_RT_TIME];
  rep->ra_events = s[S_RA_EVENTS];
  rep->ra_groups = s[S_RA_GROUPS];
  rep->ra_members = s[S_RA_EVENTS] + s[S_RA_GROUPS];
  rep->ra_bytes = s[S_RA_BYTES];
  rep->ra_time_ns = s[S_RA_TIME];
  rep->ua_events = s[S_UA_EVENTS];
  rep->ua_bytes = s[S_UA_BYTES];
  rep->ua_time_ns = s[S_UA_TIME];
  rep->ut_events = s[S_UT_EVENTS];
  rep->ut_bytes = s[S_UT_BYTES];
  rep->ut_time_ns = s[S_UT_TIME];
  rep->first_bad_event = ctl->first_bad;
  rep->status = ctl->first_bad != kNone ? 1 : 0;
  write_estimate(rep, n > rep->n_invalid, ctl->t_min, ctl->t_max, s[S_ELIM_TX] + s[S_ELIM_PAIRS]);
}
