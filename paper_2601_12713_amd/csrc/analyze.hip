// Mapping-trace analysis on gfx950 (the paper's Sec. 5, Algorithms 1-5, and
// the optimization-potential estimate of Sec. 7.6).
//
// The paper groups records with host-side maps: <hash, destination> for
// duplicates (Alg. 1), queues per <hash, destination> for round trips
// (Alg. 2), <host address, device, bytes> for repeated allocations (Alg. 3),
// a two-pointer sweep per device for unused allocations (Alg. 4) and a
// per-device kernel pointer with candidate copies for unused transfers
// (Alg. 5). Here the grouping is a stable LSD radix sort (or, for Alg. 3's
// key, a device hash table) and the per-group logic is a pass over the
// sorted order:
//
//   classify   one read of the 64-byte records: validity, per-record flags,
//              the digest sort keys, a 1-byte class / endpoint code, and
//              whether a copy-in (H2D or D2D into a device) is unused where
//              the records right after it tell
//   subsets    ordered compaction of ALLOC/DELETE, KERNEL and the other
//              copy-in records, each with its device's kernel count and
//              latest kernel end so far
//   sorts      transfers by digest (the first pass drops every other record,
//              the second the digests that occur once; low bytes first, then short runs of equal low bytes sorted in
//              place); ALLOC/DELETE by (device, device
//              address); when needed, KERNELs by (device, start) and by
//              (device, end) and copy-ins by (endpoints, source address)
//   DD/RT      forward and backward segmented scans over each digest group
//   pairing    a DELETE pairs with its predecessor in its (device, address)
//              group when that is an ALLOC; paired ALLOCs compacted in order
//   RA table   pairs grouped by (host address, device, bytes) in an
//              open-addressing table: RA = not the first pair of its key
//   UA, UT     the window [ALLOC start, DELETE end] or [copy start, next
//              copy of the place's start] against the device's kernels: from
//              the kernel counts in a chronological log, else by two binary
//              searches in the sorted kernel starts and ends
//   estimate   removable time per record over the union of its flags, the
//              log's span, the predicted speedup
//   Alg. 2     on request, the pairs the literal algorithm records
//
// Sort keys are 64-bit words; a job lists its words least significant first,
// and digit passes whose byte is the same in every key are skipped on the
// device, so the launches are fixed while the work follows the data.
#include <algorithm>
#include <cmath>
#include <cstring>

#include "internal.h"

namespace odp {
namespace {

constexpr int kT = 256;                 // threads per block
constexpr int kItems = 16;              // elements per thread in a tile
constexpr int kTile = kT * kItems;      // elements per tile
constexpr int kWaveElems = kTile / (kT / 64);  // elements per wavefront of a tile
constexpr int kRounds = kWaveElems / 64;       // rounds of 64 per wavefront
constexpr int kMaxWords = 3;
constexpr int kMaxPasses = 24;
constexpr int kEp = 11;                 // endpoints: host (0) and devices 0..9 (1..10)
constexpr uint8_t kNotTransfer = 0xFF;
// A transfer's byte beside its digest: its endpoints (device + 1 each, 0..10) as
// source * 11 + destination in the low seven bits and, in the top one, whether
// the classification found it unused. Unpacked: source << 4 | destination.
constexpr uint32_t kAuxUnused = 0x80;
__host__ __device__ inline uint32_t pack_ep(uint32_t src, uint32_t dst) { return src * kEp + dst; }
__host__ __device__ inline uint8_t unpack_ep(uint32_t a) {
  const uint32_t c = a & 0x7F, src = (c * 187) >> 11;  // c / 11 for c < 128
  return a == kNotTransfer ? kNotTransfer : (uint8_t)(src << 4 | (c - src * kEp));
}
static_assert(kEp == 11 && kEp * kEp <= 127, "a pair of endpoints in seven bits");
// Counters per wavefront of the classification, scanned into the subset
// offsets: ALLOC/DELETE, KERNEL and listed copy-in records, then KERNEL records
// per device code (device + 1).
constexpr int kWaveCnt = 3 + kEp;
// Logs of fewer than 2^24 records carry each record's endpoint byte in the
// top byte of its digest-sort value (the record index in the low 24 bits), so
// the scans over the sorted order need no gather of the code by index.
constexpr uint32_t kPackLimit = 1u << 24;
constexpr uint32_t kIdxMask = kPackLimit - 1;
constexpr uint32_t kNone = 0xFFFFFFFFu;
// Logs up to kWalkMax records are analysed by walks over all of them (below).
constexpr uint32_t kWalkMax = 4096;

// C_COPYIN: a transfer that writes device memory (H2D or D2D, dst_dev >= 0),
// the records the unused-transfer rule looks at. Logs of more than kMidMax
// records decide most of them in the classification: C_SEEN is decided but
// may be what a copy before it is searching for, C_DECIDED is neither.
enum : uint8_t { C_INVALID = 0, C_TRANSFER = 1, C_ALLOCDEL = 2, C_KERNEL = 3, C_COPYIN = 4, C_SEEN = 5, C_DECIDED = 6 };

__host__ __device__ inline uint32_t ceil_div32(uint64_t a, uint64_t b) { return (uint32_t)((a + b - 1) / b); }

// ---------------------------------------------------------------------------
// Device-side control block of one call.
// ---------------------------------------------------------------------------
struct WordMask {
  unsigned long long vor, vand;  // OR and AND over the word's values
};

struct AnaCtl {
  uint32_t n;           // records
  uint32_t n_tx;        // valid transfers (the digest sort keeps only these after its first pass)
  uint32_t n_cand;      // ... that may share their digest with another (only these after its second)
  uint32_t n_ad;        // ALLOC/DELETE records
  uint32_t n_k;         // KERNEL records
  uint32_t n_pairs;     // paired allocations
  uint32_t n_ut;        // copy-in records listed for the unused-transfer rule
  uint32_t first_bad;
  uint32_t max_ep;      // largest endpoint code among valid transfers
  WordMask m_digest, m_ad_dev, m_ad_addr, m_k_start, m_k_end, m_k_dev, m_ut_addr, m_ut_code;
  uint32_t dev_lo[kEp], dev_hi[kEp];  // per-device ranges in the sorted kernel order
  uint64_t t_min, t_max;              // earliest start and latest end of the valid records
  uint32_t kd_base[kEp], kd_total[kEp];  // KERNEL records per device code: list offsets and counts
  // wave scan tickets: blocks done per quantity, then quantities done (the
  // last user of each resets it), and each quantity's total
  uint32_t scan_tq[kWaveCnt + kEp];
  uint32_t scan_ticket;
  uint32_t plan_ticket[2];  // reductions whose last block plans a sort: blocks done
  uint64_t scan_tot[kWaveCnt + kEp];
  uint32_t ut_need_sort;              // 1: some copy-in is decided by the sorted path
  uint32_t kern_sort;                 // 1: the kernel lists are sorted (the count form's binary searches)
  // removable time (Sec. 7.6), in parts written by different stages:
  // transfers flagged DD or RT_RX; pairs flagged RA or UA; transfers flagged
  // UT only
  uint64_t elim_tx, elim_pairs;
  uint64_t ud_events, ud_bytes, ud_time;  // unused transfers by the classification's own decisions
  uint32_t wticket;                   // logs analysed by walks: workgroups done
};
constexpr int kNumMasks = 8;

// One radix sort job. 64-bit keys move with the values; a job lists its key
// words least significant first. A word with words[w] != null is gathered by
// value (words[w][value]) on the first pass that uses it; the big job's only
// word is written into keys[0] before the sort.
struct SortJob {
  const uint32_t* n_ptr;
  unsigned long long* keys[2];
  uint32_t* vals[2];
  const uint64_t* words[kMaxWords];
  const WordMask* masks[kMaxWords];
  uint32_t word_bytes[kMaxWords];  // bytes of each word that may vary
  uint32_t nwords;
  uint32_t ntiles_max;             // row length of `hist` (tiles of the capacity)
  uint32_t* hist;                  // [256][ntiles_max]
  uint32_t* totals;                // [kMaxPasses][256]
  uint32_t npasses;                // device-computed: the passes that run
  // The digest job may sort on its least significant varying bytes first
  // (np_first passes) and run each further pass (up to np_full) only when a
  // check finds a long run of equal sorted bytes holding two different keys
  // (short ones are sorted in place); other jobs: all equal.
  uint32_t np_first, np_full;
  uint8_t pw[kMaxPasses], ps[kMaxPasses];
  uint8_t pg[kMaxPasses];          // 1: this pass reads its key word from words[pw] by value
  // A word already non-decreasing in input order whenever *first_bad is kNone
  // (no record rejected), so its passes are skipped then; kNoWord if none.
  const uint32_t* first_bad;
  uint32_t mono_word;
  // When set and *run_flag is 0 the job runs no pass (its order is not needed).
  const uint32_t* run_flag;
  // 1: the classification writes the per-tile counts of the keys' least
  // significant byte, so a first pass on that byte needs no histogram launch
  uint32_t hist0_pre;
  // The digest job's first pass keeps only the valid transfers (endpoint code
  // other than kNotTransfer: in the value's top byte when *n_ptr < kPackLimit,
  // else aux[value]); the passes after it sort *n_after0 elements. Null /
  // 0 for the other jobs.
  const uint32_t* n_after0;
  const uint8_t* aux;
  uint32_t drop0;
  // The digest job's second pass keeps only the elements that may share their
  // key with another one (cand, per element of the first pass's order, from
  // sort_filter_kernel); the passes after it sort *n_after1 elements. Null:
  // no filter.
  uint8_t* cand;
  uint32_t* n_after1;
};

// Elements of job s that pass p reads.
__device__ __forceinline__ uint32_t pass_len(const SortJob& s, uint32_t p) {
  return p > 1 && s.n_after1 ? *s.n_after1 : p > 0 && s.n_after0 ? *s.n_after0 : *s.n_ptr;
}
// Elements in the job's sorted order once its passes have run (all of them
// when none ran).
__device__ __forceinline__ uint32_t sorted_len(const SortJob& s) { return pass_len(s, s.npasses); }
// Bit r: pass p of job s keeps the thread's element of round r, j0 + r * step of
// n, whose value is val[r] (used by the first pass only). The loads of all
// rounds are issued together.
template <int R>
__device__ __forceinline__ uint32_t keep_mask(const SortJob& s, uint32_t p, uint32_t j0, uint32_t step, uint32_t n,
                                              const uint32_t (&val)[R]) {
  uint32_t mask = 0;
#pragma unroll
  for (int r = 0; r < R; ++r) mask |= (uint32_t)(j0 + r * step < n) << r;
  const bool packed = *s.n_ptr < kPackLimit;
  if (p == 0 && s.drop0 && packed) {
#pragma unroll
    for (int r = 0; r < R; ++r) mask &= ~((uint32_t)((val[r] >> 24) == kNotTransfer) << r);
  } else if ((p == 0 && s.drop0) || (p == 1 && s.cand)) {
    uint8_t a[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const uint32_t j = min(j0 + r * step, n - 1);
      a[r] = p == 0 ? s.aux[j0 + r * step < n ? val[r] : 0u] : s.cand[j];
    }
    const uint8_t drop = p == 0 ? kNotTransfer : 0;
#pragma unroll
    for (int r = 0; r < R; ++r) mask &= ~((uint32_t)(a[r] == drop) << r);
  }
  return mask;
}
constexpr uint32_t kNoWord = 0xFFFFFFFFu;

struct JobSet {
  SortJob* jobs;
  uint32_t njobs;
  uint32_t stride;   // blocks per job in this launch (tiles of the call)
};

// ---------------------------------------------------------------------------
// Small helpers.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint64_t lanemask_lt() {
  const int lane = threadIdx.x & 63;
  return lane ? (~0ull >> (64 - lane)) : 0ull;
}

// Cross-lane moves on the VALU (DPP) instead of LDS permutes: the segmented
// scans below are chains of dependent moves, so their latency is what counts.
// Controls (GCN / CDNA encodings): row_shr:n, lane i of a row of 16 reads lane
// i-n of the row; row_shl:n reads lane i+n; wave_shr:1 reads lane i-1 of the
// wavefront, wave_shl:1 lane i+1. A lane whose source falls outside keeps `old`.
constexpr int kDppRowShr = 0x110, kDppRowShl = 0x100, kDppWaveShr1 = 0x138, kDppWaveShl1 = 0x130;

template <int CTRL>
__device__ __forceinline__ uint32_t dpp32(uint32_t old, uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)old, (int)x, CTRL, 0xF, 0xF, false);
}
template <int CTRL>
__device__ __forceinline__ uint64_t dpp64(uint64_t old, uint64_t x) {
  return (uint64_t)dpp32<CTRL>((uint32_t)old, (uint32_t)x) | ((uint64_t)dpp32<CTRL>((uint32_t)(old >> 32), (uint32_t)(x >> 32)) << 32);
}
__device__ __forceinline__ uint32_t lane32(uint32_t x, int l) { return (uint32_t)__builtin_amdgcn_readlane((int)x, l); }
__device__ __forceinline__ uint64_t lane64(uint64_t x, int l) {
  return (uint64_t)lane32((uint32_t)x, l) | ((uint64_t)lane32((uint32_t)(x >> 32), l) << 32);
}

__device__ __forceinline__ unsigned long long wave_sum(unsigned long long v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Sums v over the block and adds it to *dst once (dst may be null).
__device__ void block_add(uint64_t* dst64, unsigned long long v) {
  unsigned long long* dst = reinterpret_cast<unsigned long long*>(dst64);
  __shared__ unsigned long long sh[kT / 64];
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long s = 0;
    for (int w = 0; w < kT / 64; ++w) s += sh[w];
    if (s && dst) atomicAdd(dst, s);
  }
  __syncthreads();
}

// Per-block partials of the grid-wide reductions of the big launches
// (classification, subset compaction, DD/RT, RA/UA, UT): every block stores its own
// slot entry and one small kernel reduces each slot afterwards, so no two
// blocks touch the same word (same-address atomics from thousands of blocks
// serialise at one L2 channel).
enum Slot : uint32_t {
  S_N_INVALID, S_N_TRANSFERS, S_N_KERNELS, S_DIG_OR, S_DIG_AND, S_FIRST_BAD, S_MAX_EP, S_TMIN, S_TMAX,
  S_UD_EVENTS, S_UD_BYTES, S_UD_TIME,
  S_AD_DEV_OR, S_AD_DEV_AND, S_AD_ADDR_OR, S_AD_ADDR_AND, S_KS_OR, S_KS_AND, S_KE_OR, S_KE_AND, S_KD_OR, S_KD_AND,
  S_UT_ADDR_OR, S_UT_ADDR_AND, S_UT_CODE_OR, S_UT_CODE_AND,
  S_DD_EVENTS, S_DD_GROUPS, S_DD_BYTES, S_DD_TIME, S_RT_PAIRS, S_RT_RX, S_RT_BYTES, S_RT_TIME, S_ELIM_TX,
  S_RA_EVENTS, S_RA_GROUPS, S_RA_BYTES, S_RA_TIME, S_UA_EVENTS, S_UA_BYTES, S_UA_TIME, S_ELIM_PAIRS,
  S_UT_EVENTS, S_UT_BYTES, S_UT_TIME, S_ELIM_UT,
  S_PAIRS, S_UNP_ALLOC,
  kSlots
};

struct Parts {
  unsigned long long* p;  // [kSlots][stride]
  uint32_t stride;        // tiles of the capacity
  __device__ unsigned long long* at(uint32_t slot) const { return p + (size_t)slot * stride + blockIdx.x; }
};

enum RedOp : int { R_ADD, R_OR, R_AND, R_MIN, R_MAX };

template <RedOp OP>
__device__ __forceinline__ unsigned long long red2(unsigned long long a, unsigned long long b) {
  if constexpr (OP == R_ADD) return a + b;
  if constexpr (OP == R_OR) return a | b;
  if constexpr (OP == R_AND) return a & b;
  if constexpr (OP == R_MIN) return a < b ? a : b;
  return a > b ? a : b;
}

// Reduces v over the block (NT threads); thread 0 stores the result to *dst.
template <RedOp OP, int NT = kT>
__device__ void block_store(unsigned long long* dst, unsigned long long v) {
  __shared__ unsigned long long sh[NT / 64];
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v = red2<OP>(v, __shfl_xor(v, o, 64));
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long r = sh[0];
    for (int w = 1; w < NT / 64; ++w) r = red2<OP>(r, sh[w]);
    *dst = r;
  }
  __syncthreads();
}

// ---------------------------------------------------------------------------
// 0. Reset of the report and the call's counters.
// ---------------------------------------------------------------------------
// (thread t of `step`; run by the classification's launch, which reads none of it)
constexpr uint32_t kTotals = 5 * kMaxPasses * 256;  // digit totals: jobs x passes x digits
__device__ __forceinline__ void init_body(AnaCtl* ctl, odp_report* rep, uint32_t* totals, uint32_t n, uint32_t t,
                                          uint32_t step) {
  for (uint32_t i = t; i < kTotals; i += step) totals[i] = 0;
  if (t == 0) {
    unsigned long long* r = reinterpret_cast<unsigned long long*>(rep);
    for (int i = 0; i < (int)(offsetof(odp_report, predicted_speedup) / 8); ++i) r[i] = 0;
    rep->n_events = n;
    rep->predicted_speedup = 1.0;
    rep->status = 0;
    rep->first_bad_event = kNone;
    ctl->n = n;
    ctl->n_ad = ctl->n_k = ctl->n_pairs = ctl->n_ut = ctl->n_tx = ctl->n_cand = 0;
    ctl->first_bad = kNone;
    ctl->max_ep = 0;
    ctl->t_min = ~0ull;
    ctl->t_max = 0;
    ctl->elim_tx = ctl->elim_pairs = 0;
    ctl->ut_need_sort = 0;
    ctl->kern_sort = 0;
    ctl->scan_ticket = ctl->plan_ticket[0] = ctl->plan_ticket[1] = 0;
    for (int q = 0; q < kWaveCnt + kEp; ++q) ctl->scan_tq[q] = 0;
    WordMask* m = &ctl->m_digest;
    for (int i = 0; i < kNumMasks; ++i) {
      m[i].vor = 0;
      m[i].vand = ~0ull;
    }
    for (int d = 0; d < kEp; ++d) {
      ctl->dev_lo[d] = 0;
      ctl->dev_hi[d] = 0;
    }
  }
}

// An empty log: the report alone (in front of finalize_kernel).
__global__ void init_kernel(AnaCtl* ctl, odp_report* rep, uint32_t* totals) {
  init_body(ctl, rep, totals, 0, blockIdx.x * blockDim.x + threadIdx.x, gridDim.x * blockDim.x);
}

// ---------------------------------------------------------------------------
// 1. Classification: one read of every record.
// ---------------------------------------------------------------------------
__device__ __forceinline__ bool dev_ok(int d) { return d >= -1 && d <= ODP_MAX_DEVICE; }

// Hash of a key of two words (group tables, places of copies).
__device__ __forceinline__ uint32_t near_hash(uint64_t a, uint64_t b) {
  uint64_t h = (a ^ (b << 48) ^ (b >> 16)) * 0x9E3779B97F4A7C15ull;
  h ^= h >> 32;
  h *= 0xBF58476D1CE4E5B9ull;
  return (uint32_t)(h >> 32);
}

// Unused transfers inside one span of kSpanRecs consecutive records (Def. 4,
// see section 8 for the rule): most copies into device memory meet their
// device's next kernel, or the next copy to their place, a few records later,
// so the classification decides them while it holds the records, and only the
// rest is listed, gathered and searched for by the later launches. In a
// chronological log, for a copy c with no kernel still running at its start:
//   kernel k in the span   used, unless a copy to c's place lies between them
//                          and starts before k does
//   no kernel, a copy n    n starts before the span's last record does, and so
//     to the place           before any later kernel: unused
// else c is open. A copy that an open one may be looking for is the first of
// its place in its span and lies before the span's first kernel on its device,
// or is open itself (it ties with the span's last record): those are listed
// too. Kernels of earlier wavefronts that still run at c are taken into
// account at the end (ut_merge_kernel), as are logs with a rejected record,
// where none of this counts and every copy is listed.
// Starts are compared by how many records after a record start later than
// their predecessor (g below): t(a) < t(b) for a before b exactly if g(a) > g(b).
constexpr int kSpan = 8;                      // rounds of 64 records
constexpr uint32_t kSpanRecs = kSpan * 64;
constexpr uint32_t kSpanHeads = 64;
constexpr uint32_t kSpanNear = 2;
// Up to this many kernels in a round of 64 records are taken one after another,
// more by device (with every second record a kernel, 2 million of them: 394 us
// one after another, 295 by device; kernels only 441 and 294. A trace with 4 of
// 64 takes the short way.)
constexpr int kFewKernels = 8;
constexpr uint32_t kNoNode = 0xFFFFFFFFu;
constexpr uint32_t kHasPred = 1u << 31;
struct SpanLds {
  unsigned long long addr[kSpanRecs];  // source address of a copy
  uint32_t rec[kSpanRecs];             // copies: next in the bucket's chain (itself: the last) | g << 10 | endpoints << 20 | kHasPred
  uint32_t head[kSpanHeads];           // buckets by place: the node pushed last (later rounds are pushed first)
  // per device code: first the kernels counted, then (backwards) the next
  // kernel, g << 10 | record of the span, kNoNode if none
  uint32_t dev[kEp];
};
static_assert(kSpanHeads == 64 && kSpan <= 10 && kWaveElems % kSpanRecs == 0, "a head per lane, three bits per round, ten of a record of the span");

// The value of the next (previous) lane, 0 in the last (first).
__device__ __forceinline__ uint32_t wave_shl1(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x130, 0xF, 0xF, false);
}
__device__ __forceinline__ uint32_t wave_shr1(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x138, 0xF, 0xF, false);
}
// The maximum over the lanes below this one, 0 in the first.
__device__ __forceinline__ uint64_t wave_max_below(uint64_t x) {
  const int lane = threadIdx.x & 63;
  x = __shfl_up(x, 1, 64);
  if (lane == 0) x = 0;
#pragma unroll 1  // (unrolled its callers spill)
  for (int o = 1; o < 64; o <<= 1) {
    const uint64_t y = __shfl_up(x, o, 64);
    if (lane >= o) x = max(x, y);
  }
  return x;
}

// One block per tile of kTile records; wavefront w takes the 512 consecutive
// records [tile*kTile + w*512, ...), a span, in 8 rounds of 64 and also
// counts the ALLOC/DELETE, KERNEL and listed copy-in records it sees (for the
// compaction). The block also counts its tile's valid transfers by the least
// significant byte of their digest (hist0, row length ntc): the digest sort's
// first pass when that byte varies (that pass keeps only the transfers).
// Bound by the read of the records, 64 bytes each, and, for the search, by the
// latency of its LDS reads with 24 wavefronts per CU: 229 us for 10.7 million
// records (194 us without the search; by wavefronts of 16 rounds, two spans, 20
// per CU: 249, and 75 us instead of 40 at 270,000 records, where the rounds of
// a wavefront follow each other with little beside them). It leaves 3% of the
// copies to the later launches there, which took 430 us together and take 90:
// subset compaction 293 -> 69, forward search 107 -> 12, merge 30 -> 10. Spans
// of 4 rounds: 220 us, but twice the listed copies with several devices (2
// million records on 8 devices: 578 us against 503 in all). Whether a copy is
// unused travels in its sort value: DD/RT keep the flag without reading it (112
// -> 86 us).
constexpr int kClassT = kTile / kSpan;  // threads
__global__ __launch_bounds__(kClassT, 6) void classify_kernel(const odp_event* __restrict__ ev, uint32_t n, uint8_t* __restrict__ flags,
                                                         uint8_t* __restrict__ cls, uint8_t* __restrict__ aux,
                                                         unsigned long long* __restrict__ keys, uint32_t* __restrict__ vals,
                                                         uint32_t* __restrict__ wave_cnt, uint32_t* __restrict__ wave_copies,
                                                         uint64_t* __restrict__ wave_kmax, uint32_t* __restrict__ hist0,
                                                         uint32_t ntc, uint8_t* __restrict__ cand, Parts parts,
                                                         AnaCtl* ctl, odp_report* rep, uint32_t* totals) {
  init_body(ctl, rep, totals, n, blockIdx.x * kClassT + threadIdx.x, gridDim.x * kClassT);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const uint32_t wid = blockIdx.x * (kClassT / 64) + w;
  const uint32_t wb = wid * kSpanRecs;
  __shared__ unsigned long long s_kmax[kClassT / 64][kEp];
  __shared__ uint32_t s_h0[256];
  __shared__ SpanLds s_span[kClassT / 64];
  SpanLds& L = s_span[w];
  static_assert(kClassT >= 256, "one histogram bin per thread");
  if (threadIdx.x < 256) s_h0[threadIdx.x] = 0;
  L.head[lane] = kNoNode;
  if (lane < kEp) {
    L.dev[lane] = 0;
    s_kmax[w][lane] = 0;
  }
  __syncthreads();
  unsigned long long kor = 0, kand = ~0ull, tmin = ~0ull, tmax = 0;
  unsigned long long ud_b = 0, ud_t = 0;
  uint32_t n_inv = 0, n_tx = 0, bad = kNone, mep = 0, c_ad = 0, c_k = 0, c_ut = 0, c_all = 0, c_ud = 0;
  const uint64_t above = ~lanemask_lt() & ~(1ull << lane);  // lanes above this one
  // records of the next round are loaded while this round is classified; the
  // previous record of lane 0 is lane 63 of the round before
  odp_event e;
  bool in = wb + lane < n;
  if (in) e = ev[wb + lane];
  uint64_t last_prev = (lane == 0 && in && wb > 0) ? ev[wb - 1].t_start : 0;
  // of this lane's record of round r: class in bits 3r.., bit r of the others
  // whether it starts after its predecessor and what is decided of a copy
  uint32_t classes = 0, later = 0, used = 0, unused = 0;
#pragma unroll 1
  for (int r = 0; r < kSpan; ++r) {
    const uint32_t i = wb + r * 64 + lane;
    const bool in_next = r + 1 < kSpan && i + 64 < n;
    odp_event nx;
    if (in_next) nx = ev[i + 64];
    const uint64_t ts = in ? e.t_start : 0;
    uint64_t prev_start = __shfl_up(ts, 1, 64);
    if (lane == 0) prev_start = last_prev;
    last_prev = __shfl(ts, 63, 64);
    uint8_t c = C_INVALID, a = kNotTransfer;
    uint32_t dc = 0;
    if (in) {
      const bool is_tx = e.op == ODP_H2D || e.op == ODP_D2H || e.op == ODP_D2D;
      const bool valid = e.op >= ODP_ALLOC && e.op <= ODP_KERNEL && e.t_end >= e.t_start &&
                         (i == 0 || e.t_start >= prev_start) && dev_ok(e.dst_dev) && (!is_tx || dev_ok(e.src_dev));
      unsigned long long key = ~0ull;
      if (valid) {
        tmin = min(tmin, (unsigned long long)e.t_start);
        tmax = max(tmax, (unsigned long long)e.t_end);
        dc = (uint32_t)(e.dst_dev + 1);
        if (is_tx) {
          c = e.op != ODP_D2H && e.dst_dev >= 0 ? C_COPYIN : C_TRANSFER;
          a = (uint8_t)(((e.src_dev + 1) << 4) | (e.dst_dev + 1));
          mep = max(mep, (uint32_t)max(e.src_dev + 1, e.dst_dev + 1));
          key = e.digest;
          ++n_tx;
        } else if (e.op == ODP_KERNEL) {
          c = C_KERNEL;
          ++c_k;
        } else {
          c = C_ALLOCDEL;
          ++c_ad;
        }
      } else {
        ++n_inv;
        bad = min(bad, i);
      }
      if (cand) cand[i] = 1;
      keys[i] = key;
      if (c == C_TRANSFER || c == C_COPYIN) atomicAdd(&s_h0[key & 0xFF], 1u);
      kor |= key;
      kand &= key;
    }
    const bool copy = c == C_COPYIN;
    const uint64_t end = in ? e.t_end : 0;
    // a kernel of this wavefront logged before the copy still runs at its start
    uint32_t runs = copy && L.dev[dc] != 0 && s_kmax[w][dc] >= ts;
    const uint64_t kernels = __ballot(c == C_KERNEL);
    if (kernels) {
      if (__ballot(copy)) {
        if (__popcll(kernels) <= kFewKernels) {
          for (uint64_t m = kernels; m; m &= m - 1) {
            const int kl = __builtin_ctzll(m);
            const uint32_t kd = lane32(dc, kl);
            const uint64_t kend = lane64(end, kl);
            runs |= copy && lane > kl && dc == kd && kend >= ts;
          }
        } else {  // by device
          for (uint64_t m = kernels; m;) {
            const uint32_t kd = lane32(dc, __builtin_ctzll(m));
            const uint64_t on = __ballot(c == C_KERNEL && dc == kd);
            m &= ~on;
            const uint64_t latest = wave_max_below((on >> lane) & 1 ? end : 0ull);
            runs |= copy && dc == kd && (on & ~above & ~(1ull << lane)) != 0 && latest >= ts;
          }
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      if (c == C_KERNEL) {
        atomicAdd(&L.dev[dc], 1u);
        atomicMax(&s_kmax[w][dc], (unsigned long long)end);
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    classes |= (uint32_t)c << (3 * r);
    later |= (uint32_t)(in && ts > prev_start) << r;
    used |= runs << r;
    L.rec[r * 64 + lane] = (c == C_KERNEL ? dc : a) << 20;
    L.addr[r * 64 + lane] = in ? e.src_addr : 0;
    e = nx;
    in = in_next;
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  if (lane < kEp) {
    wave_cnt[kWaveCnt * wid + 3 + lane] = L.dev[lane];
    wave_kmax[kEp * wid + lane] = s_kmax[w][lane];
    L.dev[lane] = kNoNode;  // from here on the next kernel
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  // backwards: a copy joins its place's bucket and searches it
  uint32_t g_after = 0;
#pragma unroll 1
  for (int r = kSpan - 1; r >= 0; --r) {
    const uint32_t node = r * 64 + lane, c = (classes >> (3 * r)) & 7;
    const uint32_t code = L.rec[node] >> 20, dc = code & 15;
    const bool copy = c == C_COPYIN;
    const uint64_t lm = __ballot((later >> r) & 1);
    const uint32_t g = g_after + (uint32_t)__popcll(lm & above);
    // the next kernel on the receiving device
    uint32_t nk = copy ? L.dev[dc] : kNoNode;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    for (uint64_t m = __ballot(c == C_KERNEL); m;) {  // by device
      const int k0 = __builtin_ctzll(m);
      const uint32_t kd = lane32(dc, k0);
      const uint64_t on = __ballot(c == C_KERNEL && dc == kd);
      m &= ~on;
      if (copy && dc == kd && (on & above)) {
        const int kl = __builtin_ctzll(on & above);
        nk = (g_after + (uint32_t)__popcll(lm >> kl >> 1)) << 10 | (uint32_t)(r * 64 + kl);
      }
      if (lane == 0) L.dev[kd] = (g_after + (uint32_t)__popcll(lm >> k0 >> 1)) << 10 | (uint32_t)(r * 64 + k0);
    }
    const unsigned long long addr = L.addr[node];
    const uint32_t hash = near_hash(addr, code), bucket = hash % kSpanHeads;
    // The next copy of the place within kSpanNear lanes is found by lane moves, and
    // a copy that follows one so closely joins no bucket: nobody else is looking
    // for it. (A place copied to again and again had a chain of all its copies: 2
    // million copies to one place 411 us, and 279 so; two places 330 and 282. Three
    // and more take 290 either way; looking 4 lanes far cost the trace 1%.)
    const uint32_t mark = copy ? hash | 1u : 0u;
    uint32_t after = mark, before = mark, succ = 0, pred = 0;
#pragma unroll
    for (uint32_t d = 1; d <= kSpanNear; ++d) {
      after = wave_shl1(after);
      before = wave_shr1(before);
      if (copy && succ == 0 && after == mark && L.addr[node + d] == addr && L.rec[node + d] >> 20 == code) succ = d;
      if (copy && pred == 0 && before == mark && L.addr[node - d] == addr && L.rec[node - d] >> 20 == code) pred = d;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    if (copy && pred == 0) {
      const uint32_t old = atomicExch(&L.head[bucket], node);
      L.rec[node] = (old == kNoNode ? node : old) | g << 10 | code << 20;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    // the first copy to the place after this one and before that kernel. Nodes
    // of a round come in any order, rounds in order; results stay integers.
    const uint32_t limit = nk == kNoNode ? kSpanRecs : nk & 1023;
    const bool open = copy && !((used >> r) & 1);
    uint32_t best = limit, best_g = 0, cur = open && succ == 0 ? L.head[bucket] : kNoNode;
    if (open && succ != 0 && node + succ < limit) {
      best = node + succ;
      best_g = g_after + (uint32_t)__popcll(lm >> (lane + succ) >> 1);
    }
    while (__ballot(cur != kNoNode)) {
      if (cur != kNoNode) {
        const uint32_t x = L.rec[cur];
        const uint32_t hit = (uint32_t)(L.addr[cur] == addr) & (((x >> 20) & 0xFF) == code) & (cur > node) & (cur < best);
        best = hit ? cur : best;
        best_g = hit ? (x >> 10) & 1023 : best_g;
        const uint32_t nx = x & 1023;
        cur = nx == cur || (nx >> 6) > (best >> 6) ? kNoNode : nx;
      }
    }
    if (open) {
      const bool found = best != limit;
      if (found) atomicOr(&L.rec[best], kHasPred);
      const bool no = nk != kNoNode ? found && best_g > (nk >> 10) : found && best_g > 0;
      unused |= (uint32_t)no << r;
      used |= (uint32_t)(nk != kNoNode && !no) << r;
    }
    g_after += (uint32_t)__popcll(lm);
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  // classes and flags; the unused copies' bytes and durations, read again
#pragma unroll 4
  for (int r = 0; r < kSpan; ++r) {
    const uint32_t node = r * 64 + lane, i = wb + node;
    if (i < n) {
      uint8_t c = (classes >> (3 * r)) & 7;
      uint8_t f = c == C_INVALID ? ODP_F_INVALID : 0;
      const bool is_tx = c == C_TRANSFER || c == C_COPYIN;
      if (c == C_COPYIN) {
        ++c_all;
        if (((used | unused) >> r) & 1) {
          const uint32_t x = L.rec[node], first = L.dev[(x >> 20) & 15];
          const bool seen = (first == kNoNode || node < (first & 1023)) && !(x & kHasPred);
          c = seen ? C_SEEN : C_DECIDED;
        }
        c_ut += c != C_DECIDED;
      }
      if ((unused >> r) & 1) {
        f = ODP_F_UT;
        ++c_ud;
        ud_b += ev[i].bytes;
        ud_t += ev[i].t_end - ev[i].t_start;
      }
      flags[i] = f;
      cls[i] = c;
      const uint32_t ep = (L.rec[node] >> 20) & 0xFF;
      const uint32_t a = is_tx ? pack_ep(ep >> 4, ep & 15) | (f & ODP_F_UT ? kAuxUnused : 0u) : kNotTransfer;
      if (n < kPackLimit) {
        vals[i] = i | a << 24;
      } else {
        vals[i] = i;
        aux[i] = (uint8_t)a;
      }
    }
  }
  const uint32_t n_k = c_k;
  // per-wavefront subset counts
  for (int o = 32; o >= 1; o >>= 1) {
    c_ad += __shfl_xor(c_ad, o, 64);
    c_k += __shfl_xor(c_k, o, 64);
    c_ut += __shfl_xor(c_ut, o, 64);
    c_all += __shfl_xor(c_all, o, 64);
  }
  if (lane == 0) {
    wave_cnt[kWaveCnt * wid] = c_ad;
    wave_cnt[kWaveCnt * wid + 1] = c_k;
    wave_cnt[kWaveCnt * wid + 2] = c_ut;
    wave_copies[wid] = c_all;
  }
  __syncthreads();
  if (threadIdx.x < 256) hist0[(size_t)threadIdx.x * ntc + blockIdx.x] = s_h0[threadIdx.x];
  block_store<R_ADD, kClassT>(parts.at(S_N_INVALID), n_inv);
  block_store<R_ADD, kClassT>(parts.at(S_N_TRANSFERS), n_tx);
  block_store<R_ADD, kClassT>(parts.at(S_N_KERNELS), n_k);
  block_store<R_OR, kClassT>(parts.at(S_DIG_OR), kor);
  block_store<R_AND, kClassT>(parts.at(S_DIG_AND), kand);
  block_store<R_MIN, kClassT>(parts.at(S_FIRST_BAD), bad);
  block_store<R_MAX, kClassT>(parts.at(S_MAX_EP), mep);
  block_store<R_MIN, kClassT>(parts.at(S_TMIN), tmin);
  block_store<R_MAX, kClassT>(parts.at(S_TMAX), tmax);
  block_store<R_ADD, kClassT>(parts.at(S_UD_EVENTS), c_ud);
  block_store<R_ADD, kClassT>(parts.at(S_UD_BYTES), ud_b);
  block_store<R_ADD, kClassT>(parts.at(S_UD_TIME), ud_t);
}

// ---------------------------------------------------------------------------
// 2. Ordered compaction of the ALLOC/DELETE and KERNEL subsets.
// ---------------------------------------------------------------------------
// Exclusive scan of K interleaved u32 counters (cnt[K*t + c]) over `ntiles`
// entries (one block, for short arrays); the totals of the first two go to
// tot0 / tot1 where not null.
template <int K>
__global__ __launch_bounds__(1024) void scan_counts_kernel(uint32_t* cnt, uint32_t ntiles, uint32_t* tot0,
                                                           uint32_t* tot1) {
  __shared__ uint32_t wsum[K][16];
  __shared__ uint32_t carry[K];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (threadIdx.x < K) carry[threadIdx.x] = 0;
  __syncthreads();
  for (uint32_t base = 0; base < ntiles; base += 1024) {
    const uint32_t t = base + threadIdx.x;
    uint32_t own[K], x[K];
#pragma unroll
    for (int c = 0; c < K; ++c) {
      own[c] = t < ntiles ? cnt[K * t + c] : 0;
      x[c] = own[c];
      for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(x[c], o, 64);
        if (lane >= o) x[c] += y;
      }
      if (lane == 63) wsum[c][w] = x[c];
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < K; ++c) {
      uint32_t before = carry[c] + x[c] - own[c];
      for (int q = 0; q < w; ++q) before += wsum[c][q];
      if (t < ntiles) cnt[K * t + c] = before;
    }
    __syncthreads();
    if (threadIdx.x < K) {
      uint32_t s = 0;
      for (int q = 0; q < 16; ++q) s += wsum[threadIdx.x][q];
      carry[threadIdx.x] += s;
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    if (tot0) *tot0 = carry[0];
    if (K > 1 && tot1) *tot1 = carry[K > 1 ? 1 : 0];
  }
}

// The classification's per-wavefront counters (kWaveCnt sums) and per-device
// latest kernel ends (kEp maxima), scanned into exclusive prefixes in two
// steps: each block of 1,024 wavefronts scans its chunk in place and stores
// the chunk's totals; one block then scans the chunk totals (the consumer adds
// its chunk's prefix). Rounds of 1,024 entries, one thread each, so every
// load is coalesced.
struct WaveScan {
  uint32_t* cnt;   // [nw][kWaveCnt]
  uint64_t* kmax;  // [nw][kEp]
  uint32_t* ccnt;  // [nchunk][kWaveCnt]: chunk totals, then their exclusive prefixes
  uint64_t* cmax;  // [nchunk][kEp]
  uint32_t nw;
  // [nw], or null: all copy-ins of the wavefronts, counted instead of the
  // listed ones (cnt[..][2]) in a log with a rejected record
  const uint32_t* copies;
};
constexpr uint32_t kScanChunk = 1024;

// Exclusive scans of the per-wavefront counts (kWaveCnt, sums) and maxima
// (kEp) in one launch: block (q, c) scans quantity q over chunk c of
// kScanChunk wavefronts; the last block of a quantity, by a ticket, scans the
// quantity's chunk totals, and the last quantity to finish writes the subset
// sizes and per-device kernel list offsets. One quantity per block keeps the
// kernel's code short: it runs once per call, from cold instruction caches,
// where a block holding every quantity at once (unrolled) took 30 us.
constexpr int kScanQ = kWaveCnt + kEp;

// Exclusive scan of x over the 1024 threads of the block (sum, or max when
// MAX); returns the prefix and sets total. wt: 16 words of LDS.
template <typename T, bool MAX>
__device__ __forceinline__ T block_xscan(T x, T* wt, T& total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  T v = x;
  for (int o = 1; o < 64; o <<= 1) {
    const T y = __shfl_up(v, o, 64);
    if (lane >= o) v = MAX ? max(v, y) : v + y;
  }
  if (lane == 63) wt[w] = v;
  __syncthreads();
  if (w == 0) {
    T u = lane < 16 ? wt[lane] : (T)0;
    for (int o = 1; o < 16; o <<= 1) {
      const T y = __shfl_up(u, o, 64);
      if (lane >= o) u = MAX ? max(u, y) : u + y;
    }
    if (lane < 16) wt[lane] = u;  // inclusive over wavefronts
  }
  __syncthreads();
  T before = __shfl_up(v, 1, 64);
  if (lane == 0) before = 0;
  const T wb = w > 0 ? wt[w - 1] : (T)0;
  total = wt[15];
  __syncthreads();  // wt is reused by the next scan
  return MAX ? max(wb, before) : wb + before;
}

// Scans quantity q (element i at base[stride * i]) over [c * kScanChunk, ...)
// in place (from the values instead[i] when given); then the quantity's chunk totals (ct[stride * c]) by its last
// block. Returns true in the block that finished the quantity last overall.
template <typename T, bool MAX>
__device__ bool scan_quantity(T* base, T* ct, uint32_t stride, uint32_t nw, uint32_t nchunk, uint32_t c, uint32_t q,
                              AnaCtl* ctl, T* wt, uint32_t* flag, const T* instead = nullptr) {
  const uint32_t i = c * kScanChunk + threadIdx.x;
  const bool in = i < nw;
  T total;
  const T x = block_xscan<T, MAX>(in ? instead ? instead[i] : base[(size_t)stride * i] : (T)0, wt, total);
  if (in) base[(size_t)stride * i] = x;
  // the chunk total reaches the device-coherent level before the ticket:
  // an agent-scope store and a wait for its completion, not a fence (an
  // agent-scope fence writes back the L2)
  if (threadIdx.x == 0) {
    __hip_atomic_store(ct + (size_t)stride * c, total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    *flag = __hip_atomic_fetch_add(&ctl->scan_tq[q], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == nchunk - 1;
  }
  __syncthreads();
  if (!*flag) return false;
  T carry = 0;
  for (uint32_t b0 = 0; b0 < nchunk; b0 += kScanChunk) {
    const uint32_t k = b0 + threadIdx.x;
    const bool ok = k < nchunk;
    const T y = ok ? __hip_atomic_load(ct + (size_t)stride * k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : (T)0;
    T t;
    const T e = block_xscan<T, MAX>(y, wt, t);
    if (ok) ct[(size_t)stride * k] = MAX ? max(carry, e) : carry + e;
    carry = MAX ? max(carry, t) : carry + t;
  }
  if (threadIdx.x == 0) {
    ctl->scan_tq[q] = 0;
    __hip_atomic_store(&ctl->scan_tot[q], (uint64_t)carry, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    *flag = __hip_atomic_fetch_add(&ctl->scan_ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == kScanQ - 1;
  }
  __syncthreads();
  return *flag != 0;
}

__device__ void wave_scan_body(const WaveScan& S, uint32_t nchunk, AnaCtl* ctl) {
  __shared__ unsigned long long wt[16];
  __shared__ uint32_t flag;
  const uint32_t q = blockIdx.x / nchunk, c = blockIdx.x % nchunk;
  const bool last =
      q < kWaveCnt
          ? scan_quantity<uint32_t, false>(S.cnt + q, S.ccnt + q, kWaveCnt, S.nw, nchunk, c, q, ctl,
                                           reinterpret_cast<uint32_t*>(wt), &flag,
                                           q == 2 && S.copies && ctl->first_bad != kNone ? S.copies : nullptr)
          : scan_quantity<unsigned long long, true>(reinterpret_cast<unsigned long long*>(S.kmax) + (q - kWaveCnt),
                                                    reinterpret_cast<unsigned long long*>(S.cmax) + (q - kWaveCnt), kEp,
                                                    S.nw, nchunk, c, q, ctl, wt, &flag);
  if (!last || threadIdx.x != 0) return;
  uint64_t tot[kWaveCnt];
  for (int k = 0; k < kWaveCnt; ++k)
    tot[k] = __hip_atomic_load(&ctl->scan_tot[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  ctl->scan_ticket = 0;
  ctl->n_ad = (uint32_t)tot[0];
  ctl->n_k = (uint32_t)tot[1];
  ctl->n_ut = (uint32_t)tot[2];
  uint32_t b = 0;
  for (int d = 0; d < kEp; ++d) {
    ctl->kd_base[d] = b;
    ctl->kd_total[d] = (uint32_t)tot[3 + d];
    b += (uint32_t)tot[3 + d];
  }
}

__global__ __launch_bounds__(1024) void wave_scan_kernel(WaveScan S, uint32_t nchunk, AnaCtl* ctl) {
  wave_scan_body(S, nchunk, ctl);
}

constexpr uint8_t kUtSeen = 4;
struct SubsetOut {
  uint32_t* ut_idx;     // listed copy-ins: record index
  uint64_t* ut_w_addr;  // source address
  uint64_t* ut_w_code;  // endpoint code (src_dev + 1) << 4 | (dst_dev + 1)
  uint64_t* ut_ts;      // t_start
  uint32_t* ut_vals;
  uint32_t* ut_kc;      // KERNEL records on the receiving device logged before the copy
  uint64_t* ut_km;      // the latest end among those (0 when there is none)
  uint8_t* ut_hit;      // kUtSeen for a copy that is decided already (C_SEEN)
  uint32_t* ad_kc;      // ALLOC/DELETE: KERNEL records on its device logged before it
  uint64_t* ad_km;      // ... and the latest end among them
  uint64_t* kd_ts;      // KERNEL records per device code in log order (from kd_base[code]): start
  uint32_t* kd_idx;     // ... and record index
  const AnaCtl* ctl;
  uint32_t* ad_idx;
  uint8_t* ad_op;
  uint64_t* ad_w_dev;
  uint64_t* ad_w_addr;
  uint32_t* ad_vals;
  uint32_t* ad_alloc_partner;
  uint32_t* k_idx;
  uint64_t* k_w_start;
  uint64_t* k_w_end;
  uint64_t* k_w_dev;
  uint32_t* k_vals_s;
  uint32_t* k_vals_e;
};

// Ordered compaction of the ALLOC/DELETE, KERNEL and copy-in records. Wavefront w
// takes 1,024 records: it first gathers which of them are listed (of the copy-ins
// those the classification left open, or all in a log with a rejected record)
// in record order, then reads those, 64 at a time (one record in eight in the
// trace workload; by 16 rounds of all records: 170 us instead of 69 for 10.7
// million). A ballot per round gives each matching lane its rank, so the
// entries land in record order at the wavefront's scanned offsets, and the
// records of a round are read together. Each copy-in also gets the number of
// KERNEL records on its receiving device logged before it: the device's count
// before the wavefront (scanned) plus the kernels of earlier rounds and lanes.
// ROUNDS rounds per wavefront. MID (logs of up to kMidMax records): no sort
// words, values and masks are written, but each ALLOC/DELETE's host address and
// bytes, and the kernels' ends in their per-device lists.
template <int ROUNDS, bool MID>
__device__ void subset_scatter_body(const odp_event* __restrict__ ev, const uint8_t* __restrict__ cls, uint32_t n,
                                    const WaveScan& W, const SubsetOut& S, const Parts& parts, uint64_t* ad_host,
                                    uint64_t* ad_bytes, uint64_t* kd_te) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const uint32_t wid = blockIdx.x * (kT / 64) + w;
  const uint32_t wb = wid * (ROUNDS * 64);
  uint8_t c[ROUNDS];
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const uint32_t i = wb + r * 64 + lane;
    c[r] = i < n ? cls[i] : C_INVALID;
  }
  const uint64_t lt = lanemask_lt();
  const uint8_t last_ut = !MID && S.ctl->first_bad != kNone ? C_DECIDED : C_SEEN;
  // the listed records of the wavefront: class << 10 | record
  __shared__ uint16_t s_list[MID ? 1 : kT / 64][MID ? 1 : ROUNDS * 64];
  uint32_t rounds = ROUNDS, listed = 0;
  if constexpr (!MID) {
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
      const bool take = c[r] >= C_ALLOCDEL && c[r] <= last_ut;
      const uint64_t m = __ballot(take);
      if (take) s_list[w][listed + (uint32_t)__popcll(m & lt)] = (uint16_t)((uint32_t)c[r] << 10 | (uint32_t)(r * 64 + lane));
      listed += (uint32_t)__popcll(m);
    }
    rounds = ceil_div32(listed, 64);
  }
  // offsets: the wavefront's prefix within its chunk plus the chunk's prefix
  const uint32_t ent = MID ? wid : wb / kSpanRecs;
  const uint32_t* wo = W.cnt + (size_t)kWaveCnt * ent;
  const uint32_t* co = W.ccnt + (size_t)kWaveCnt * (ent / kScanChunk);
  uint32_t q0 = wo[0] + co[0], q1 = wo[1] + co[1], q2 = wo[2] + co[2];
  __shared__ uint32_t s_kc[kT / 64][kEp];            // kernels per device code before the current round
  __shared__ unsigned long long s_km[kT / 64][kEp];  // the latest end among them
  if (lane < kEp) {
    s_kc[w][lane] = wo[3 + lane] + co[3 + lane];
    s_km[w][lane] = max((unsigned long long)W.kmax[(size_t)kEp * ent + lane],
                        (unsigned long long)W.cmax[(size_t)kEp * (ent / kScanChunk) + lane]);
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  unsigned long long o_dev = 0, a_dev = ~0ull, o_addr = 0, a_addr = ~0ull, o_ks = 0, a_ks = ~0ull, o_ke = 0,
                     a_ke = ~0ull, o_kd = 0, a_kd = ~0ull, o_ua = 0, a_ua = ~0ull, o_uc = 0, a_uc = ~0ull;
  constexpr int kUnroll = MID ? ROUNDS : 2;
#pragma unroll kUnroll
  for (uint32_t r = 0; r < rounds; ++r) {
    uint32_t i = wb + r * 64 + lane, cr = C_INVALID;
    if constexpr (MID) {
      cr = c[r];
    } else if (r * 64 + lane < listed) {
      const uint32_t x = s_list[w][r * 64 + lane];
      i = wb + (x & 1023);
      cr = x >> 10;
    }
    const bool is_ad = cr == C_ALLOCDEL, is_k = cr == C_KERNEL;
    const bool is_ut = cr >= C_COPYIN && cr <= last_ut;
    const uint64_t bad = __ballot(is_ad), bk = __ballot(is_k), bu = __ballot(is_ut);
    // the whole record, once, for the records this kernel lists
    odp_event e{};
    if (is_k || is_ut || is_ad) e = ev[i];
    // the device code of kernels and copy-ins (both in dst_dev)
    const uint32_t dc = (is_k || is_ut || is_ad) ? (uint32_t)(e.dst_dev + 1) : 0u;
    const unsigned long long kend = is_k ? (unsigned long long)e.t_end : 0ull;
    uint32_t kc = (is_ut || is_k || is_ad) ? s_kc[w][dc] : 0u;
    unsigned long long km = (is_ut || is_ad) ? s_km[w][dc] : 0ull;
    if (bk) {
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      if (__popcll(bk) <= kFewKernels) {
        for (uint64_t m = bk; m; m &= m - 1) {  // this round's kernels, one after another
          const int kl = __builtin_ctzll(m);
          const uint32_t d = lane32(dc, kl);
          const unsigned long long te = lane64(kend, kl);
          const uint32_t on = dc == d && lane > kl;
          kc += on;
          km = on ? max(km, te) : km;
        }
      } else {  // by device
        for (uint64_t m = bk; m;) {
          const uint32_t d = lane32(dc, __builtin_ctzll(m));
          const uint64_t on = __ballot(is_k && dc == d);
          m &= ~on;
          if (dc == d) kc += (uint32_t)__popcll(on & lt);
          if (!__ballot((is_ut || is_ad) && dc == d)) continue;
          const unsigned long long latest = wave_max_below((on >> lane) & 1 ? kend : 0ull);
          if (dc == d) km = max(km, latest);
        }
      }
      if (is_k) {
        atomicAdd(&s_kc[w][dc], 1u);
        atomicMax(&s_km[w][dc], kend);
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    if (is_ut) {
      const uint32_t q = q2 + (uint32_t)__popcll(bu & lt);
      const uint64_t code = (uint64_t)(((e.src_dev + 1) << 4) | (e.dst_dev + 1)), sa = e.src_addr;
      S.ut_idx[q] = i;
      S.ut_w_addr[q] = sa;
      S.ut_w_code[q] = code;
      S.ut_ts[q] = e.t_start;
      S.ut_vals[q] = MID ? near_hash(sa, code) : q;  // MID: a hash of the place
      S.ut_kc[q] = kc;
      S.ut_km[q] = km;
      if constexpr (!MID) S.ut_hit[q] = cr == C_SEEN ? kUtSeen : 0;
      o_ua |= sa;
      a_ua &= sa;
      o_uc |= code;
      a_uc &= code;
    } else if (is_ad) {
      const uint32_t q = q0 + (uint32_t)__popcll(bad & lt);
      const uint64_t dv = (uint64_t)(e.dst_dev + 1), ad = e.dst_addr;
      S.ad_idx[q] = i;
      S.ad_op[q] = e.op;
      S.ad_w_dev[q] = dv;
      S.ad_w_addr[q] = ad;
      if constexpr (MID) {
        ad_host[q] = e.src_addr;
        ad_bytes[q] = e.bytes;
      } else {
        S.ad_vals[q] = q;
      }
      S.ad_alloc_partner[q] = kNone;
      S.ad_kc[q] = kc;
      S.ad_km[q] = km;
      o_dev |= dv;
      a_dev &= dv;
      o_addr |= ad;
      a_addr &= ad;
    } else if (is_k) {
      const uint32_t q = q1 + (uint32_t)__popcll(bk & lt);
      const uint64_t dv = (uint64_t)(e.dst_dev + 1);
      if constexpr (!MID) {
        S.k_idx[q] = i;
        S.k_w_start[q] = e.t_start;
        S.k_w_end[q] = e.t_end;
        S.k_w_dev[q] = dv;
        S.k_vals_s[q] = q;
        S.k_vals_e[q] = q;
      }
      // this kernel's place among its device's kernels in log order
      const uint32_t kp = S.ctl->kd_base[dc] + kc;
      S.kd_ts[kp] = e.t_start;
      S.kd_idx[kp] = i;
      if constexpr (MID) kd_te[kp] = e.t_end;
      o_ks |= e.t_start;
      a_ks &= e.t_start;
      o_ke |= e.t_end;
      a_ke &= e.t_end;
      o_kd |= dv;
      a_kd &= dv;
    }
    q0 += (uint32_t)__popcll(bad);
    q1 += (uint32_t)__popcll(bk);
    q2 += (uint32_t)__popcll(bu);
  }
  if constexpr (MID) return;
  // (identity values where a lane saw no such record)
  block_store<R_OR>(parts.at(S_AD_DEV_OR), o_dev);
  block_store<R_AND>(parts.at(S_AD_DEV_AND), a_dev);
  block_store<R_OR>(parts.at(S_AD_ADDR_OR), o_addr);
  block_store<R_AND>(parts.at(S_AD_ADDR_AND), a_addr);
  block_store<R_OR>(parts.at(S_KS_OR), o_ks);
  block_store<R_AND>(parts.at(S_KS_AND), a_ks);
  block_store<R_OR>(parts.at(S_KE_OR), o_ke);
  block_store<R_AND>(parts.at(S_KE_AND), a_ke);
  block_store<R_OR>(parts.at(S_KD_OR), o_kd);
  block_store<R_AND>(parts.at(S_KD_AND), a_kd);
  block_store<R_OR>(parts.at(S_UT_ADDR_OR), o_ua);
  block_store<R_AND>(parts.at(S_UT_ADDR_AND), a_ua);
  block_store<R_OR>(parts.at(S_UT_CODE_OR), o_uc);
  block_store<R_AND>(parts.at(S_UT_CODE_AND), a_uc);
}

__global__ __launch_bounds__(kT) void subset_scatter_kernel(const odp_event* ev, const uint8_t* cls, uint32_t n, WaveScan W,
                                                            SubsetOut S, Parts parts) {
  subset_scatter_body<kRounds, false>(ev, cls, n, W, S, parts, nullptr, nullptr, nullptr);
}

// A store that another block of the same launch may read (all_read) once it
// has seen the ticket drawn after it: at agent scope, since the XCDs' L2s do
// not see each other's stores.
template <typename T>
__device__ __forceinline__ void to_all(T* p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ T all_read(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One block per slot: reduces the blocks' partials of slots [first, first +
// gridDim.x) into the control block and the report.
template <int NT>
__device__ void reduce_slot(const Parts& parts, uint32_t nb, uint32_t slot, AnaCtl* ctl, odp_report* rep) {
  const unsigned long long* p = parts.p + (size_t)slot * parts.stride;
  int op = R_ADD;
  switch (slot) {
    case S_DIG_OR: case S_AD_DEV_OR: case S_AD_ADDR_OR: case S_KS_OR: case S_KE_OR: case S_KD_OR:
    case S_UT_ADDR_OR: case S_UT_CODE_OR: op = R_OR; break;
    case S_DIG_AND: case S_AD_DEV_AND: case S_AD_ADDR_AND: case S_KS_AND: case S_KE_AND: case S_KD_AND:
    case S_UT_ADDR_AND: case S_UT_CODE_AND: op = R_AND; break;
    case S_FIRST_BAD: case S_TMIN: op = R_MIN; break;
    case S_MAX_EP: case S_TMAX: op = R_MAX; break;
    default: break;
  }
  unsigned long long v = op == R_AND || op == R_MIN ? ~0ull : 0ull;
  for (uint32_t b = threadIdx.x; b < nb; b += NT) {
    const unsigned long long x = p[b];
    v = op == R_ADD ? v + x : op == R_OR ? (v | x) : op == R_AND ? (v & x) : op == R_MIN ? min(v, x) : max(v, x);
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    const unsigned long long x = __shfl_xor(v, o, 64);
    v = op == R_ADD ? v + x : op == R_OR ? (v | x) : op == R_AND ? (v & x) : op == R_MIN ? min(v, x) : max(v, x);
  }
  __shared__ unsigned long long sh[NT / 64];
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x != 0) return;
  for (int t = 1; t < NT / 64; ++t) {
    const unsigned long long x = sh[t];
    v = op == R_ADD ? v + x : op == R_OR ? (v | x) : op == R_AND ? (v & x) : op == R_MIN ? min(v, x) : max(v, x);
  }
  switch (slot) {
    case S_N_INVALID: rep->n_invalid = v; break;
    case S_N_TRANSFERS:
      rep->n_transfers = v;
      ctl->n_tx = (uint32_t)v;
      break;
    case S_N_KERNELS: rep->n_kernels = v; break;
    case S_DIG_OR: to_all(&ctl->m_digest.vor, v); break;
    case S_DIG_AND: to_all(&ctl->m_digest.vand, v); break;
    case S_FIRST_BAD: to_all(&ctl->first_bad, (uint32_t)min(v, (unsigned long long)kNone)); break;
    case S_MAX_EP: ctl->max_ep = (uint32_t)v; break;
    case S_TMIN: ctl->t_min = v; break;
    case S_TMAX: ctl->t_max = v; break;
    case S_UD_EVENTS: ctl->ud_events = v; break;
    case S_UD_BYTES: ctl->ud_bytes = v; break;
    case S_UD_TIME: ctl->ud_time = v; break;
    case S_UT_ADDR_OR: to_all(&ctl->m_ut_addr.vor, v); break;
    case S_UT_ADDR_AND: to_all(&ctl->m_ut_addr.vand, v); break;
    case S_UT_CODE_OR: to_all(&ctl->m_ut_code.vor, v); break;
    case S_UT_CODE_AND: to_all(&ctl->m_ut_code.vand, v); break;
    case S_ELIM_TX: ctl->elim_tx = v; break;
    case S_AD_DEV_OR: to_all(&ctl->m_ad_dev.vor, v); break;
    case S_AD_DEV_AND: to_all(&ctl->m_ad_dev.vand, v); break;
    case S_AD_ADDR_OR: to_all(&ctl->m_ad_addr.vor, v); break;
    case S_AD_ADDR_AND: to_all(&ctl->m_ad_addr.vand, v); break;
    case S_KS_OR: to_all(&ctl->m_k_start.vor, v); break;
    case S_KS_AND: to_all(&ctl->m_k_start.vand, v); break;
    case S_KE_OR: to_all(&ctl->m_k_end.vor, v); break;
    case S_KE_AND: to_all(&ctl->m_k_end.vand, v); break;
    case S_KD_OR: to_all(&ctl->m_k_dev.vor, v); break;
    case S_KD_AND: to_all(&ctl->m_k_dev.vand, v); break;
    case S_DD_EVENTS: rep->dd_events = v; break;
    case S_DD_GROUPS: rep->dd_groups = v; break;
    case S_DD_BYTES: rep->dd_bytes = v; break;
    case S_DD_TIME: rep->dd_time_ns = v; break;
    case S_RT_PAIRS: rep->rt_pairs = v; break;
    case S_RT_RX: rep->rt_rx_events = v; break;
    case S_RT_BYTES: rep->rt_bytes = v; break;
    case S_RT_TIME: rep->rt_time_ns = v; break;
    case S_RA_EVENTS: rep->ra_events = v; break;
    case S_RA_GROUPS: rep->ra_groups = v; break;
    case S_RA_BYTES: rep->ra_bytes = v; break;
    case S_RA_TIME: rep->ra_time_ns = v; break;
    case S_UA_EVENTS: rep->ua_events = v; break;
    case S_UA_BYTES: rep->ua_bytes = v; break;
    case S_UA_TIME: rep->ua_time_ns = v; break;
    case S_ELIM_PAIRS: ctl->elim_pairs = v; break;
    default: break;
  }
}

// ---------------------------------------------------------------------------
// 3. LSD radix sort, 8-bit digits, several independent jobs per launch.
// ---------------------------------------------------------------------------
// What a reduction's last block plans: the jobs' passes, from the masks that the
// reduction has just written (njobs 0: nothing). first_passes: when nonzero, the
// passes after that many are deferred to the local fix (digest job only).
// cand, n_after1: the filter's arrays for the job, or null to run without it.
struct PlanArgs {
  JobSet J;
  uint32_t first_passes;
  uint8_t* cand;
  uint32_t* n_after1;
  uint32_t* ticket;
};

__device__ void sort_plan(SortJob& s, const PlanArgs& P) {
  s.cand = P.cand;
  s.n_after1 = P.n_after1;
  uint32_t np = 0;
  const uint32_t skip = (s.first_bad && all_read(s.first_bad) == kNone) ? s.mono_word : kNoWord;
  const uint32_t nwords = (s.run_flag && *s.run_flag == 0) ? 0u : s.nwords;
  for (uint32_t w = 0; w < nwords; ++w) {
    if (w == skip) continue;
    // bits that are 1 in some key and 0 in another (0 when there are no keys)
    const unsigned long long var = all_read(&s.masks[w]->vor) & ~all_read(&s.masks[w]->vand);
    bool first = true;
    for (uint32_t b = 0; b < s.word_bytes[w]; ++b)
      if ((var >> (8 * b)) & 0xFF) {
        s.pw[np] = (uint8_t)w;
        s.ps[np] = (uint8_t)(8 * b);
        s.pg[np] = (uint8_t)(first && s.words[w] != nullptr);
        first = false;
        ++np;
      }
  }
  s.np_full = np;
  s.np_first = P.first_passes ? min(np, P.first_passes) : np;
  s.npasses = s.np_first;
}

__global__ __launch_bounds__(kT) void reduce_parts_kernel(Parts parts, uint32_t nb, uint32_t first, AnaCtl* ctl,
                                                          odp_report* rep, PlanArgs P) {
  reduce_slot<kT>(parts, nb, first + blockIdx.x, ctl, rep);
  if (P.J.njobs == 0) return;
  __shared__ uint32_t s_last;
  if (threadIdx.x == 0) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    s_last = __hip_atomic_fetch_add(P.ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1;
  }
  __syncthreads();
  if (s_last && threadIdx.x < P.J.njobs) sort_plan(P.J.jobs[threadIdx.x], P);
}

// Local fix of the digest job, launched before the first deferred pass
// (p = np_first: the check) and once after the last (p = kFixFinal: the
// sort). After the passes 0..p-1, the keys, sorted stably on those bytes, fall
// into runs of equal sorted bytes. The duplicate and round-trip scans need
// each digest's elements together and in input order only, so a run that
// holds one digest is done, and a run that holds several (which may
// interleave) is done once sorted stably by the whole key. A run longer than
// kFixMax that holds several digests switches every remaining pass on (the
// full stable sort then leaves nothing to fix); otherwise the short runs are
// sorted in place after the (skipped) passes.
//
// Check (npasses == p): a "collision" is an element whose key differs from its
// predecessor's in the same run. Each block stages a tile of kFixTile keys with
// kFixHalo more on each side in LDS, which holds every key a walk of at most
// kFixMax steps reaches. The first collision of each run walks to the run's
// ends and records the run (start << 32 | length) in the buffers pass p would
// write: tile t keeps its count in vals[(p+1)&1][t] and its runs at
// keys[(p+1)&1][t * kFixTile/2 ...]; a tile holds at most kFixTile/2 first
// collisions, since each has its run's previous element before it. No key
// moves in the check, so every walk sees the same array.
// Sort (p = kFixFinal, npasses == np_first < np_full, so the check found no
// long run and no deferred pass ran): a block per tile of the check, a thread
// per recorded run, each an insertion sort; the runs are disjoint.
constexpr uint32_t kFixMax = 128;
constexpr uint32_t kFixFinal = 0xFFFFFFFFu;
constexpr uint32_t kFixTile = 4 * kT;
constexpr uint32_t kFixHalo = kFixMax + 1;
constexpr uint32_t kWalkIdle = 0, kWalking = 1, kWalkEnd = 2, kWalkLong = 3;

__global__ __launch_bounds__(kT) void sort_fix_kernel(SortJob* job, uint32_t p) {
  SortJob& s = *job;
  // One read per block: a check that finds a long run raises npasses while
  // other blocks of the same launch start, and every wavefront of a block
  // must take the same branch (the check's barriers).
  __shared__ uint32_t s_np;
  if (threadIdx.x == 0) s_np = __hip_atomic_load(&s.npasses, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  const uint32_t np = s_np;
  const uint32_t n = pass_len(s, s.np_first);  // the sorted elements
  const uint32_t nft = (n + kFixTile - 1) / kFixTile;
  if (p == kFixFinal) {
    if (np != s.np_first || np >= s.np_full) return;
    const uint32_t q = np;  // the pass the check ran before
    const unsigned long long* runs = s.keys[(q + 1) & 1];
    const uint32_t* cnt = s.vals[(q + 1) & 1];
    unsigned long long* k = s.keys[q & 1];
    uint32_t* v = s.vals[q & 1];
    for (uint32_t t = blockIdx.x; t < nft; t += gridDim.x) {
      const uint32_t c = cnt[t];
      for (uint32_t r = threadIdx.x; r < c; r += kT) {
        const unsigned long long run = runs[(size_t)t * (kFixTile / 2) + r];
        const uint32_t j = (uint32_t)(run >> 32), e = j + (uint32_t)run;
        for (uint32_t a = j + 1; a < e; ++a) {  // stable: equal keys keep their order
          const unsigned long long ka = k[a];
          const uint32_t va = v[a];
          uint32_t b = a;
          while (b > j && k[b - 1] > ka) {
            k[b] = k[b - 1];
            v[b] = v[b - 1];
            --b;
          }
          k[b] = ka;
          v[b] = va;
        }
      }
    }
    return;
  }
  if (np != p || p >= s.np_full) return;
  unsigned long long mask = 0;
  for (uint32_t q = 0; q < p; ++q) mask |= 0xFFull << s.ps[q];
  const unsigned long long* k = s.keys[p & 1];
  unsigned long long* runs = s.keys[(p + 1) & 1];
  uint32_t* cnt = s.vals[(p + 1) & 1];
  __shared__ unsigned long long s_k[kFixTile + 2 * kFixHalo];
  __shared__ uint32_t s_w[kT / 64];
  const uint32_t lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  bool long_mixed = false;
  for (uint32_t t = blockIdx.x; t < nft; t += gridDim.x) {
    // s_k[i] holds key lo + i (where 0 <= lo + i < n)
    const long long lo = (long long)t * kFixTile - kFixHalo;
    for (uint32_t i = threadIdx.x; i < kFixTile + 2 * kFixHalo; i += kT) {
      const long long g = lo + i;
      if (g >= 0 && g < (long long)n) s_k[i] = k[g];
    }
    __syncthreads();
    uint32_t recorded = 0;
    for (uint32_t r = 0; r < kFixTile / kT; ++r) {
      const uint32_t j = t * kFixTile + r * kT + threadIdx.x;
      // Both walks loop while any lane of the wavefront still walks, so all
      // lanes leave them together and their outcome is a plain integer
      // (hipcc has lost per-lane booleans set in a loop that lanes leave at
      // different trips).
      uint32_t st = 0, e = 0, back = kWalkIdle, fwd = kWalkIdle;
      unsigned long long kj = 0, kp = 0;
      if (j > 0 && j < n) {
        kj = s_k[j - lo];
        kp = s_k[j - 1 - lo];
        if (kj != kp && ((kj ^ kp) & mask) == 0) {
          st = j - 1;
          back = kWalking;
        }
      }
      // back to the run's start st (every key in [st, j) equals kp), or to
      // an earlier collision
      while (__ballot(back == kWalking)) {
        if (back == kWalking) {
          if (j - st >= kFixMax) {
            back = kWalkLong;
          } else if (st == 0) {
            back = kWalkEnd;
          } else {
            const unsigned long long c = s_k[st - 1 - lo];
            if (((c ^ kj) & mask) != 0) back = kWalkEnd;
            else if (c != kp) back = kWalkIdle;  // not the run's first collision
            else --st;
          }
        }
      }
      // forward to the run's end e (exclusive)
      if (back == kWalkEnd) {
        e = j + 1;
        fwd = kWalking;
      }
      while (__ballot(fwd == kWalking)) {
        if (fwd == kWalking) {
          if (e - st > kFixMax) fwd = kWalkLong;
          else if (e >= n || ((s_k[e - lo] ^ kj) & mask) != 0) fwd = kWalkEnd;
          else ++e;
        }
      }
      long_mixed |= back == kWalkLong || fwd == kWalkLong;
      const bool rec = fwd == kWalkEnd;
      const uint64_t m = __ballot(rec);
      if (lane == 0) s_w[w] = (uint32_t)__popcll(m);
      __syncthreads();
      uint32_t off = recorded, tot = 0;
      for (uint32_t q = 0; q < kT / 64; ++q) {
        off += q < w ? s_w[q] : 0u;
        tot += s_w[q];
      }
      if (rec)
        runs[(size_t)t * (kFixTile / 2) + off + (uint32_t)__popcll(m & lanemask_lt())] =
            ((unsigned long long)st << 32) | (e - st);
      recorded += tot;
      __syncthreads();
    }
    if (threadIdx.x == 0) cnt[t] = recorded;
  }
  if (__syncthreads_or(long_mixed) && threadIdx.x == 0) s.npasses = s.np_full;
}

// Locates this block's job and first tile; returns false when the block has
// no work in pass p. A job's blocks (J.stride of them) take its tiles
// tile, tile + stride, ... (next_tile), so a launch may have fewer blocks per
// job than the job has tiles.
__device__ __forceinline__ bool job_tile(const JobSet& J, uint32_t p, const SortJob*& s, uint32_t& tile, uint32_t& n) {
  const uint32_t j = blockIdx.x / J.stride;
  if (j >= J.njobs) return false;
  const SortJob& c = J.jobs[j];
  s = &c;
  tile = blockIdx.x % J.stride;
  n = pass_len(c, p);
  return p < c.npasses && (uint64_t)tile * kTile < n && tile < c.ntiles_max;
}
__device__ __forceinline__ bool next_tile(const JobSet& J, const SortJob* s, uint32_t& tile, uint32_t n) {
  tile += J.stride;
  return (uint64_t)tile * kTile < n && tile < s->ntiles_max;
}

// Counts the digits of a tile. All loads of a thread are issued before any is
// waited for (a load under its element's condition, one after another, took
// 35 us instead of 22 for the 9.8 million elements of the trace's second pass,
// and 13 instead of 8 for the 2 million of its third).
__global__ __launch_bounds__(kT) void sort_hist_kernel(JobSet J, uint32_t p) {
  const SortJob* s;
  uint32_t tile, n;
  if (!job_tile(J, p, s, tile, n)) return;
  if (p == 0 && s->hist0_pre && s->ps[0] == 0) return;  // counted by the classification
  __shared__ uint32_t h[256];
  do {
  h[threadIdx.x] = 0;
  __syncthreads();
  const uint32_t src = p & 1;
  const uint32_t b = tile * kTile;
  const uint32_t shift = s->ps[p];
  const bool gather = s->pg[p] != 0;  // the keys are read from the pass's word by value, else carried
  uint32_t val[kItems];
  unsigned long long key[kItems];
  if (gather || p == 0) {
#pragma unroll
    for (int r = 0; r < kItems; ++r) val[r] = s->vals[src][min(b + r * kT + threadIdx.x, n - 1)];
  }
  if (gather) {
    const uint64_t* word = s->words[s->pw[p]];
#pragma unroll
    for (int r = 0; r < kItems; ++r) key[r] = word[val[r]];
  } else {
#pragma unroll
    for (int r = 0; r < kItems; ++r) key[r] = s->keys[src][min(b + r * kT + threadIdx.x, n - 1)];
  }
  const uint32_t mask = keep_mask(*s, p, b + threadIdx.x, kT, n, val);
#pragma unroll
  for (int r = 0; r < kItems; ++r)
    if ((mask >> r) & 1) atomicAdd(&h[(uint32_t)(key[r] >> shift) & 0xFF], 1u);
  __syncthreads();
  s->hist[threadIdx.x * s->ntiles_max + tile] = h[threadIdx.x];
  __syncthreads();
  } while (next_tile(J, s, tile, n));
}

// One block per (job, digit): exclusive scan of the digit's row over tiles;
// the row total goes to totals[pass][digit] (the scatter adds the counts of
// smaller digits). Each thread sums a run of consecutive tiles, the runs are
// scanned across the block, then written back.
__global__ __launch_bounds__(kT) void sort_scan_kernel(JobSet J, uint32_t p) {
  const uint32_t j = blockIdx.x / 256, d = blockIdx.x % 256;
  if (j >= J.njobs) return;
  const SortJob& s = J.jobs[j];
  if (p >= s.npasses) return;
  const uint32_t n = pass_len(s, p);
  const uint32_t nt = ceil_div32(n, kTile);
  __shared__ uint32_t wsum[kT / 64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  uint32_t* row = s.hist + (size_t)d * s.ntiles_max;
  const uint32_t per = ceil_div32(nt, kT);
  const uint32_t t0 = threadIdx.x * per, t1 = min(nt, t0 + per);
  uint32_t run = 0;
  for (uint32_t t = t0; t < t1; ++t) run += row[t];
  uint32_t x = run;
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) wsum[w] = x;
  __syncthreads();
  uint32_t before = 0;
  for (int q = 0; q < w; ++q) before += wsum[q];
  before += x - run;
  for (uint32_t t = t0; t < t1; ++t) {
    const uint32_t c = row[t];
    row[t] = before;
    before += c;
  }
  if (threadIdx.x == kT - 1) {
    s.totals[p * 256 + d] = before;
    if (p == 1 && s.n_after1 && before) atomicAdd(s.n_after1, before);
  }
}

// Stable scatter, 512 threads per tile (twice the wavefronts of the other
// sort kernels, for latency hiding at this kernel's LDS footprint). Each
// wavefront ranks its 512 consecutive elements (8 rounds of 64) by digit with
// ballots; the tile is then placed in digit order in LDS and written out in
// that order, so the global writes form one contiguous run per digit.
constexpr int kST = 512;                      // threads of the scatter
constexpr int kSW = kST / 64;                 // its wavefronts
constexpr int kSElems = kTile / kSW;          // elements per wavefront
constexpr int kSRounds = kSElems / 64;        // rounds of 64 per wavefront

__global__ __launch_bounds__(kST) void sort_scatter_kernel(JobSet J, uint32_t p) {
  const SortJob* s;
  uint32_t tile, n;
  if (!job_tile(J, p, s, tile, n)) return;
  __shared__ uint32_t wcnt[kSW][256];
  __shared__ uint32_t lbase[256];   // tile-local start of each digit
  __shared__ uint32_t gbase[256];   // global start of each digit's run of this tile
  __shared__ unsigned long long stage[kTile];
  __shared__ uint8_t sdig[kTile];
  __shared__ uint32_t ws[4], wt[4];
  __shared__ uint32_t s_kept;       // elements of this tile the pass writes
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  do {
  for (int x = 0; x < 256; x += 64) wcnt[w][x + lane] = 0;
  __syncthreads();
  const uint32_t src = p & 1, dst = src ^ 1;
  const uint32_t tb = tile * kTile;
  const uint32_t wb = tb + w * kSElems;
  const uint32_t shift = s->ps[p];
  const bool gather = s->pg[p] != 0;
  const uint64_t* word = s->words[s->pw[p]];
  uint32_t dg[kSRounds], rk[kSRounds], vl[kSRounds];
  unsigned long long ky[kSRounds];
#pragma unroll
  for (int r = 0; r < kSRounds; ++r) {
    const uint32_t j = wb + r * 64 + lane;
    const bool in = j < n;
    vl[r] = in ? s->vals[src][j] : 0u;
    ky[r] = (in && !gather) ? s->keys[src][j] : 0ull;
  }
  if (gather) {
#pragma unroll
    for (int r = 0; r < kSRounds; ++r) {
      const uint32_t j = wb + r * 64 + lane;
      if (j < n) ky[r] = word[vl[r]];
    }
  }
  // bit r: this lane's element of round r is written by the pass
  const uint32_t inmask = keep_mask(*s, p, wb + lane, 64, n, vl);
#pragma unroll
  for (int r = 0; r < kSRounds; ++r) {
    const bool in = (inmask >> r) & 1;
    const uint32_t d = in ? (uint32_t)(ky[r] >> shift) & 0xFF : 0u;
    uint64_t peers = __ballot(in);
#pragma unroll
    for (int bit = 0; bit < 8; ++bit) {
      const uint64_t bb = __ballot((d >> bit) & 1);
      peers &= ((d >> bit) & 1) ? bb : ~bb;
    }
    const uint32_t before = in ? wcnt[w][d] : 0;
    const uint32_t cnt = __popcll(peers);
    const bool leader = in && (peers >> lane) == 1ull;  // highest lane among peers
    dg[r] = d;
    rk[r] = before + (uint32_t)__popcll(peers & lanemask_lt());
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    if (leader) wcnt[w][d] = before + cnt;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  }
  __syncthreads();
  if (threadIdx.x < 256) {
    // per digit (threads 0..255): counts of the wavefronts before, tile-local and global bases
    const uint32_t d = threadIdx.x;
    uint32_t c = 0;
    for (int x = 0; x < kSW; ++x) {
      const uint32_t t = wcnt[x][d];
      wcnt[x][d] = c;
      c += t;
    }
    // exclusive scan of the tile counts over digits
    uint32_t xsc = c;
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t y = __shfl_up(xsc, o, 64);
      if (lane >= o) xsc += y;
    }
    if (lane == 63) ws[w] = xsc;
    // global start: counts of smaller digits over all tiles, plus earlier tiles of this digit
    const uint32_t tot = s->totals[p * 256 + d];
    uint32_t y = tot;
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t z = __shfl_up(y, o, 64);
      if (lane >= o) y += z;
    }
    if (lane == 63) wt[w] = y;
    lbase[d] = xsc - c;  // completed below with the sums of earlier wavefronts
    gbase[d] = y - tot + s->hist[(size_t)d * s->ntiles_max + tile];
    if (d == 255) s_kept = c;
  }
  __syncthreads();
  if (threadIdx.x < 256) {
    const uint32_t d = threadIdx.x;
    uint32_t pre = 0, gpre = 0;
    for (int q = 0; q < w; ++q) {
      pre += ws[q];
      gpre += wt[q];
    }
    lbase[d] += pre;
    gbase[d] += gpre;
    if (d == 255) s_kept += lbase[255];
  }
  __syncthreads();
  const uint32_t cnt_tile = s_kept;
  // pass 1: values (and digits) into tile-local digit order
#pragma unroll
  for (int r = 0; r < kSRounds; ++r) {
    if ((inmask >> r) & 1) {
      const uint32_t lp = lbase[dg[r]] + wcnt[w][dg[r]] + rk[r];
      reinterpret_cast<uint32_t*>(stage)[lp] = vl[r];
      sdig[lp] = (uint8_t)dg[r];
    }
  }
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < cnt_tile; i += kST) {
    const uint32_t d = sdig[i];
    s->vals[dst][gbase[d] + (i - lbase[d])] = reinterpret_cast<uint32_t*>(stage)[i];
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kSRounds; ++r)
    if ((inmask >> r) & 1) stage[lbase[dg[r]] + wcnt[w][dg[r]] + rk[r]] = ky[r];
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < cnt_tile; i += kST) {
    const uint32_t d = sdig[i];
    s->keys[dst][gbase[d] + (i - lbase[d])] = stage[i];
  }
  __syncthreads();
  } while (next_tile(J, s, tile, n));
}

// Between the digest job's first two passes: marks the transfers that may share
// their digest with another one. A transfer whose digest no other carries is no
// duplicate, no round trip and no group, and in a log where most content is
// moved once (8.1 of the 9.8 million transfers of the trace workload) those are
// most of the elements that the later passes, the fix and the scans would carry.
// Equal digests lie in one digit's range of the first pass's order: a workgroup
// takes a range and keeps two bits per hash of a digest in LDS, "occurs" and
// "occurs again". Two digests that share a hash are only kept for nothing (7% of
// the single ones at 38,500 per range and 2^19 hashes). A range of more than
// kFilterMax elements (one digest moved again and again, or more than 33
// million transfers) keeps all of its elements, as the classification marked
// them: there are few single digests in it to drop, or too many for the bits.
// Bound by the read of the keys and the LDS atomics: 30 us for the 9.8 million
// transfers of the 10.7-million-record trace, where it takes 7.9 million
// elements out of the second and third pass, the fix and the scans (the whole
// analysis 1,409 -> 1,215 us).
constexpr uint32_t kFilterT = 1024;
constexpr uint32_t kFilterBits = 19;
constexpr uint32_t kFilterMax = 1u << 17;
constexpr int kFilterHeld = 40;  // elements per thread held in registers between the two steps

__device__ __forceinline__ uint32_t filter_hash(unsigned long long key) {
  return (uint32_t)((key * 0x9E3779B97F4A7C15ull) >> (64 - kFilterBits));
}

__global__ __launch_bounds__(kFilterT) void sort_filter_kernel(SortJob* job) {
  SortJob& s = *job;
  __shared__ uint32_t s_once[1u << (kFilterBits - 5)], s_again[1u << (kFilterBits - 5)];
  __shared__ uint32_t s_lo, s_len;
  if (s.npasses < 2) return;
  const uint32_t t = threadIdx.x;
  // the range of digit blockIdx.x
  if (t < 64) {
    uint32_t before = 0;
    for (uint32_t d = t; d < blockIdx.x; d += 64) before += s.totals[d];
    before = (uint32_t)wave_sum(before);
    if (t == 0) {
      s_lo = before;
      s_len = s.totals[blockIdx.x];
    }
  }
  __syncthreads();
  const uint32_t lo = s_lo, len = s_len;
  if (len == 0 || len > kFilterMax) return;
  for (uint32_t x = t; x < (1u << (kFilterBits - 5)); x += kFilterT) s_once[x] = s_again[x] = 0;
  __syncthreads();
  const unsigned long long* k = s.keys[1] + lo;
  uint8_t* cand = s.cand + lo;
  auto mark = [&](uint32_t h) {
    const uint32_t bit = 1u << (h & 31);
    if (atomicOr(&s_once[h >> 5], bit) & bit) atomicOr(&s_again[h >> 5], bit);
  };
  uint32_t held[kFilterHeld];
#pragma unroll
  for (int u = 0; u < kFilterHeld; ++u) {
    held[u] = 0;
    if ((uint32_t)u * kFilterT < len) {
      const uint32_t j = (uint32_t)u * kFilterT + t;
      if (j < len) held[u] = filter_hash(k[j]);
    }
  }
#pragma unroll
  for (int u = 0; u < kFilterHeld; ++u)
    if ((uint32_t)u * kFilterT + t < len) mark(held[u]);
  for (uint32_t j = kFilterHeld * kFilterT + t; j < len; j += kFilterT) mark(filter_hash(k[j]));
  __syncthreads();
#pragma unroll
  for (int u = 0; u < kFilterHeld; ++u) {
    const uint32_t j = (uint32_t)u * kFilterT + t;
    if (j < len) cand[j] = (uint8_t)((s_again[held[u] >> 5] >> (held[u] & 31)) & 1);
  }
  for (uint32_t j = kFilterHeld * kFilterT + t; j < len; j += kFilterT) {
    const uint32_t h = filter_hash(k[j]);
    cand[j] = (uint8_t)((s_again[h >> 5] >> (h & 31)) & 1);
  }
}

// ---------------------------------------------------------------------------
// 4. Duplicate and round-trip transfers: segmented scans per digest group.
//
// Over the digest-sorted order (index order inside a group), the forward
// state of a record is what the earlier transfers of its group hold: the
// receivers seen and, per unordered endpoint pair, whether it occurred and the
// direction of its latest transfer. The backward state is what the later
// transfers hold: the ordered pairs and receivers seen.
//   DD     my receiver is in the forward receivers
//   RT_RX  my pair occurred earlier and its latest transfer went the other way
//   RT_TX  the reverse of my ordered pair occurs later
//   group  a record that is not DD but whose receiver occurs later starts a
//          duplicate group (dd_groups)
// Two state widths: one 32-bit word when only endpoint codes 0..3 occur (host
// and devices 0..2), five words for all 11 endpoints.
// ---------------------------------------------------------------------------
template <int MODE>
struct FS;  // forward state
template <int MODE>
struct BS;  // backward state

// Small: endpoints 0..3. Forward: bits 0-3 receivers, 4-9 pair present,
// 10-15 pair direction. Backward: bits 0-3 receivers, 4-15 ordered pairs.
template <>
struct FS<0> {
  uint32_t w;
};
template <>
struct BS<0> {
  uint32_t w;
};
// General: endpoints 0..10.
template <>
struct FS<1> {
  uint32_t dst;
  uint64_t pres, dir;
};
template <>
struct BS<1> {
  uint32_t dst;
  uint64_t lo, hi;
};

// Unordered pair (lo < hi) of E endpoints -> 0 .. E(E-1)/2 - 1.
__device__ __forceinline__ uint32_t upair(uint32_t lo, uint32_t hi, uint32_t E) {
  return lo * (2 * E - lo - 1) / 2 + (hi - lo - 1);
}
// Ordered pair (s != d) -> 0 .. E(E-1) - 1.
__device__ __forceinline__ uint32_t opair(uint32_t s, uint32_t d, uint32_t E) {
  return s * (E - 1) + (d < s ? d : d - 1);
}

template <int MODE>
struct St;

template <>
struct St<0> {
  static constexpr uint32_t E = 4;
  __device__ static FS<0> fid() { return FS<0>{0}; }
  __device__ static BS<0> bid() { return BS<0>{0}; }
  __device__ static FS<0> flift(uint8_t a) {
    if (a == kNotTransfer) return fid();
    const uint32_t s = a >> 4, d = a & 15;
    uint32_t w = 1u << d;
    if (s != d) {
      const uint32_t lo = min(s, d), hi = max(s, d), u = upair(lo, hi, E);
      w |= 1u << (4 + u);
      if (s == lo) w |= 1u << (10 + u);
    }
    return FS<0>{w};
  }
  __device__ static BS<0> blift(uint8_t a) {
    if (a == kNotTransfer) return bid();
    const uint32_t s = a >> 4, d = a & 15;
    uint32_t w = 1u << d;
    if (s != d) w |= 1u << (4 + opair(s, d, E));
    return BS<0>{w};
  }
  // a earlier, b later
  __device__ static FS<0> fop(FS<0> a, FS<0> b) {
    const uint32_t bp = (b.w >> 4) & 0x3F;
    const uint32_t keep = ~(bp << 10);
    return FS<0>{((a.w & keep) | b.w)};
  }
  __device__ static BS<0> bop(BS<0> a, BS<0> b) { return BS<0>{a.w | b.w}; }
  __device__ static bool has_dst(FS<0> f, uint32_t d) { return (f.w >> d) & 1; }
  __device__ static bool has_dst(BS<0> b, uint32_t d) { return (b.w >> d) & 1; }
  __device__ static bool rx(FS<0> f, uint32_t s, uint32_t d) {
    const uint32_t lo = min(s, d), hi = max(s, d), u = upair(lo, hi, E);
    return ((f.w >> (4 + u)) & 1) && (((f.w >> (10 + u)) & 1) != (s == lo));
  }
  __device__ static bool tx(BS<0> b, uint32_t s, uint32_t d) { return (b.w >> (4 + opair(d, s, E))) & 1; }
  __device__ static FS<0> shfl_up(FS<0> x, int o) { return FS<0>{(uint32_t)__shfl_up((int)x.w, o, 64)}; }
  __device__ static BS<0> shfl_down(BS<0> x, int o) { return BS<0>{(uint32_t)__shfl_down((int)x.w, o, 64)}; }
  __device__ static FS<0> shfl(FS<0> x, int l) { return FS<0>{(uint32_t)__shfl((int)x.w, l, 64)}; }
  __device__ static BS<0> shfl(BS<0> x, int l) { return BS<0>{(uint32_t)__shfl((int)x.w, l, 64)}; }
  template <int C>
  __device__ static FS<0> dpp(FS<0> old, FS<0> x) { return FS<0>{dpp32<C>(old.w, x.w)}; }
  template <int C>
  __device__ static BS<0> dpp(BS<0> old, BS<0> x) { return BS<0>{dpp32<C>(old.w, x.w)}; }
  __device__ static FS<0> lane(FS<0> x, int l) { return FS<0>{lane32(x.w, l)}; }
  __device__ static BS<0> lane(BS<0> x, int l) { return BS<0>{lane32(x.w, l)}; }
};

template <>
struct St<1> {
  static constexpr uint32_t E = kEp;
  __device__ static FS<1> fid() { return FS<1>{0, 0, 0}; }
  __device__ static BS<1> bid() { return BS<1>{0, 0, 0}; }
  __device__ static FS<1> flift(uint8_t a) {
    if (a == kNotTransfer) return fid();
    const uint32_t s = a >> 4, d = a & 15;
    FS<1> f{1u << d, 0, 0};
    if (s != d) {
      const uint32_t lo = min(s, d), hi = max(s, d), u = upair(lo, hi, E);
      f.pres = 1ull << u;
      if (s == lo) f.dir = 1ull << u;
    }
    return f;
  }
  __device__ static BS<1> blift(uint8_t a) {
    if (a == kNotTransfer) return bid();
    const uint32_t s = a >> 4, d = a & 15;
    BS<1> b{1u << d, 0, 0};
    if (s != d) {
      const uint32_t o = opair(s, d, E);
      if (o < 64) b.lo = 1ull << o; else b.hi = 1ull << (o - 64);
    }
    return b;
  }
  __device__ static FS<1> fop(const FS<1>& a, const FS<1>& b) {
    return FS<1>{a.dst | b.dst, a.pres | b.pres, (a.dir & ~b.pres) | b.dir};
  }
  __device__ static BS<1> bop(const BS<1>& a, const BS<1>& b) { return BS<1>{a.dst | b.dst, a.lo | b.lo, a.hi | b.hi}; }
  __device__ static bool has_dst(const FS<1>& f, uint32_t d) { return (f.dst >> d) & 1; }
  __device__ static bool has_dst(const BS<1>& b, uint32_t d) { return (b.dst >> d) & 1; }
  __device__ static bool rx(const FS<1>& f, uint32_t s, uint32_t d) {
    const uint32_t lo = min(s, d), hi = max(s, d), u = upair(lo, hi, E);
    return ((f.pres >> u) & 1) && (((f.dir >> u) & 1) != (s == lo));
  }
  __device__ static bool tx(const BS<1>& b, uint32_t s, uint32_t d) {
    const uint32_t o = opair(d, s, E);
    return o < 64 ? ((b.lo >> o) & 1) : ((b.hi >> (o - 64)) & 1);
  }
  __device__ static FS<1> shfl_up(const FS<1>& x, int o) {
    return FS<1>{(uint32_t)__shfl_up((int)x.dst, o, 64), __shfl_up(x.pres, o, 64), __shfl_up(x.dir, o, 64)};
  }
  __device__ static BS<1> shfl_down(const BS<1>& x, int o) {
    return BS<1>{(uint32_t)__shfl_down((int)x.dst, o, 64), __shfl_down(x.lo, o, 64), __shfl_down(x.hi, o, 64)};
  }
  __device__ static FS<1> shfl(const FS<1>& x, int l) {
    return FS<1>{(uint32_t)__shfl((int)x.dst, l, 64), __shfl(x.pres, l, 64), __shfl(x.dir, l, 64)};
  }
  __device__ static BS<1> shfl(const BS<1>& x, int l) {
    return BS<1>{(uint32_t)__shfl((int)x.dst, l, 64), __shfl(x.lo, l, 64), __shfl(x.hi, l, 64)};
  }
  template <int C>
  __device__ static FS<1> dpp(const FS<1>& old, const FS<1>& x) {
    return FS<1>{dpp32<C>(old.dst, x.dst), dpp64<C>(old.pres, x.pres), dpp64<C>(old.dir, x.dir)};
  }
  template <int C>
  __device__ static BS<1> dpp(const BS<1>& old, const BS<1>& x) {
    return BS<1>{dpp32<C>(old.dst, x.dst), dpp64<C>(old.lo, x.lo), dpp64<C>(old.hi, x.hi)};
  }
  __device__ static FS<1> lane(const FS<1>& x, int l) { return FS<1>{lane32(x.dst, l), lane64(x.pres, l), lane64(x.dir, l)}; }
  __device__ static BS<1> lane(const BS<1>& x, int l) { return BS<1>{lane32(x.dst, l), lane64(x.lo, l), lane64(x.hi, l)}; }
};

// Carry records per wavefront (1,024 consecutive sorted elements).
struct WaveAgg {
  uint32_t ff, bf;   // a group starts (forward) / ends (backward) inside the wavefront
  uint32_t fs[5];    // forward state since the last start
  uint32_t bs[5];    // backward state up to the first end
};

template <int MODE>
__device__ __forceinline__ void put_f(uint32_t* w, const FS<MODE>& f);
template <int MODE>
__device__ __forceinline__ FS<MODE> get_f(const uint32_t* w);
template <int MODE>
__device__ __forceinline__ void put_b(uint32_t* w, const BS<MODE>& b);
template <int MODE>
__device__ __forceinline__ BS<MODE> get_b(const uint32_t* w);
template <>
__device__ __forceinline__ void put_f<0>(uint32_t* w, const FS<0>& f) { w[0] = f.w; }
template <>
__device__ __forceinline__ FS<0> get_f<0>(const uint32_t* w) { return FS<0>{w[0]}; }
template <>
__device__ __forceinline__ void put_b<0>(uint32_t* w, const BS<0>& b) { w[0] = b.w; }
template <>
__device__ __forceinline__ BS<0> get_b<0>(const uint32_t* w) { return BS<0>{w[0]}; }
template <>
__device__ __forceinline__ void put_f<1>(uint32_t* w, const FS<1>& f) {
  w[0] = f.dst;
  w[1] = (uint32_t)f.pres;
  w[2] = (uint32_t)(f.pres >> 32);
  w[3] = (uint32_t)f.dir;
  w[4] = (uint32_t)(f.dir >> 32);
}
template <>
__device__ __forceinline__ FS<1> get_f<1>(const uint32_t* w) {
  return FS<1>{w[0], (uint64_t)w[1] | ((uint64_t)w[2] << 32), (uint64_t)w[3] | ((uint64_t)w[4] << 32)};
}
template <>
__device__ __forceinline__ void put_b<1>(uint32_t* w, const BS<1>& b) {
  w[0] = b.dst;
  w[1] = (uint32_t)b.lo;
  w[2] = (uint32_t)(b.lo >> 32);
  w[3] = (uint32_t)b.hi;
  w[4] = (uint32_t)(b.hi >> 32);
}
template <>
__device__ __forceinline__ BS<1> get_b<1>(const uint32_t* w) {
  return BS<1>{w[0], (uint64_t)w[1] | ((uint64_t)w[2] << 32), (uint64_t)w[3] | ((uint64_t)w[4] << 32)};
}

struct DDArgs {
  const odp_event* ev;
  uint32_t n;          // records of the log (values are packed when n < kPackLimit)
  const uint8_t* aux;
  const SortJob* job;  // the digest job (keys/vals in buffer npasses & 1)
  const AnaCtl* ctl;
  WaveAgg* agg;        // per wavefront
  WaveAgg* carry;      // per wavefront: forward carry-in / backward carry-in
  uint8_t* flags;
  odp_report* rep;
  Parts parts;
  const uint8_t* uth;  // per record: 1 for an unused transfer (logs of up to kMidMax records; else null)
};


// Inclusive segmented scans inside one round of 64 lanes: (f, v) pairs where
// f marks a segment start at or before the lane (forward) or a segment end at
// or after it (backward). Four DPP steps scan each row of 16 lanes; the row
// totals, read into scalars, then carry across rows.
template <int MODE, int CTRL>
__device__ __forceinline__ void fstep(uint32_t& f, FS<MODE>& v) {
  using S = St<MODE>;
  const uint32_t fo = dpp32<CTRL>(0u, f);
  const FS<MODE> vo = S::template dpp<CTRL>(S::fid(), v);
  if (!f) v = S::fop(vo, v);
  f |= fo;
}
template <int MODE, int CTRL>
__device__ __forceinline__ void bstep(uint32_t& f, BS<MODE>& v) {
  using S = St<MODE>;
  const uint32_t fo = dpp32<CTRL>(0u, f);
  const BS<MODE> vo = S::template dpp<CTRL>(S::bid(), v);
  if (!f) v = S::bop(v, vo);
  f |= fo;
}
template <int MODE>
__device__ __forceinline__ void wave_fscan(uint32_t& f, FS<MODE>& v) {
  using S = St<MODE>;
  fstep<MODE, kDppRowShr + 1>(f, v);
  fstep<MODE, kDppRowShr + 2>(f, v);
  fstep<MODE, kDppRowShr + 4>(f, v);
  fstep<MODE, kDppRowShr + 8>(f, v);
  // prefixes of rows 1..3: the totals of the rows before, in order
  uint32_t pf = lane32(f, 15);
  FS<MODE> pv = S::lane(v, 15);
  const uint32_t f31 = lane32(f, 31), f47 = lane32(f, 47);
  const FS<MODE> v31 = S::lane(v, 31), v47 = S::lane(v, 47);
  const int row = (threadIdx.x & 63) >> 4;
  if (row >= 2) {
    pv = f31 ? v31 : S::fop(pv, v31);
    pf |= f31;
  }
  if (row == 3) {
    pv = f47 ? v47 : S::fop(pv, v47);
    pf |= f47;
  }
  if (row >= 1) {
    if (!f) v = S::fop(pv, v);
    f |= pf;
  }
}
template <int MODE>
__device__ __forceinline__ void wave_bscan(uint32_t& f, BS<MODE>& v) {
  using S = St<MODE>;
  bstep<MODE, kDppRowShl + 1>(f, v);
  bstep<MODE, kDppRowShl + 2>(f, v);
  bstep<MODE, kDppRowShl + 4>(f, v);
  bstep<MODE, kDppRowShl + 8>(f, v);
  // suffixes of rows 0..2: the totals of the rows after, in order
  uint32_t qf = lane32(f, 48);
  BS<MODE> qv = S::lane(v, 48);
  const uint32_t f32 = lane32(f, 32), f16 = lane32(f, 16);
  const BS<MODE> v32 = S::lane(v, 32), v16 = S::lane(v, 16);
  const int row = (threadIdx.x & 63) >> 4;
  if (row <= 1) {
    qv = f32 ? v32 : S::bop(v32, qv);
    qf |= f32;
  }
  if (row == 0) {
    qv = f16 ? v16 : S::bop(v16, qv);
    qf |= f16;
  }
  if (row <= 2) {
    if (!f) v = S::bop(v, qv);
    f |= qf;
  }
}

// Orders this wavefront's LDS writes before its later LDS reads by other lanes.
__device__ __forceinline__ void wave_lds_fence() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

// Elements of the digest job's sorted order the scans read.
__device__ __forceinline__ uint32_t dd_len(const DDArgs& A) { return sorted_len(*A.job); }

// All 16 rounds of a wavefront at once: keys and values (coalesced), then
// the endpoint codes gathered by value, all loads in flight together. Values
// and codes go to the wavefront's LDS rows; bit r of heads / tails says
// whether this lane's element of round r starts / ends its digest group, of
// unused whether the classification found it unused.
// n: the sorted elements; packed: codes in the values' top byte.
template <int ROUNDS>
__device__ __forceinline__ void load_wave(const unsigned long long* k, const uint32_t* v, const uint8_t* aux,
                                          uint32_t n, bool packed, uint32_t wb, uint32_t* s_val, uint8_t* s_code,
                                          uint32_t& heads, uint32_t& tails, uint32_t& unused) {
  const int lane = threadIdx.x & 63;
  unsigned long long key[ROUNDS];
  uint32_t val[ROUNDS];
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const uint32_t j = wb + r * 64 + lane;
    key[r] = j < n ? k[j] : 0ull;
    val[r] = j < n ? v[j] : 0u;
  }
  const unsigned long long before = (lane == 0 && wb > 0 && wb < n) ? k[wb - 1] : 0ull;
  const unsigned long long after = (lane == 63 && wb + (ROUNDS * 64) < n) ? k[wb + (ROUNDS * 64)] : 0ull;
  uint8_t a[ROUNDS];
  if (packed) {
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
      a[r] = wb + r * 64 + lane < n ? (uint8_t)(val[r] >> 24) : kNotTransfer;
      val[r] &= kIdxMask;
    }
  } else {
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) a[r] = wb + r * 64 + lane < n ? aux[val[r]] : kNotTransfer;
  }
  heads = tails = unused = 0;
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const uint32_t j = wb + r * 64 + lane;
    const bool in = j < n;
    unsigned long long prev = __shfl_up(key[r], 1, 64);
    unsigned long long next = __shfl_down(key[r], 1, 64);
    const unsigned long long last_before = r > 0 ? __shfl(key[r > 0 ? r - 1 : 0], 63, 64) : before;
    const unsigned long long first_after = r + 1 < ROUNDS ? __shfl(key[r + 1 < ROUNDS ? r + 1 : r], 0, 64) : after;
    if (lane == 0) prev = last_before;
    if (lane == 63) next = first_after;
    heads |= (uint32_t)(in && (j == 0 || prev != key[r])) << r;
    tails |= (uint32_t)(in && (j + 1 == n || next != key[r])) << r;
    s_val[r * 64 + lane] = val[r];
    s_code[r * 64 + lane] = unpack_ep(a[r]);
    unused |= (uint32_t)(a[r] != kNotTransfer && (a[r] & kAuxUnused)) << r;
  }
  wave_lds_fence();
}

// One round of 64 sorted elements: endpoint code (gathered by value) and
// whether the element starts / ends its digest group.
__device__ __forceinline__ void load_round(const unsigned long long* k, const uint32_t* v, const uint8_t* aux,
                                           uint32_t n, bool packed, uint32_t j, uint8_t& a, bool& head, bool& tail) {
  const int lane = threadIdx.x & 63;
  const bool in = j < n;
  const unsigned long long key = in ? k[j] : 0ull;
  unsigned long long prev = __shfl_up(key, 1, 64);
  unsigned long long next = __shfl_down(key, 1, 64);
  if (lane == 0 && in && j > 0) prev = k[j - 1];
  if (lane == 63 && in && j + 1 < n) next = k[j + 1];
  head = in && (j == 0 || prev != key);
  tail = in && (j + 1 == n || next != key);
  a = !in ? kNotTransfer : unpack_ep(packed ? v[j] >> 24 : aux[v[j]]);
}

// Per-wavefront aggregates. The forward one folds the elements after the
// wavefront's last group start, the backward one those before its first
// group end, so rounds are read from each end only until such a boundary
// turns up (one round each for typical groups; all 16 for a group that
// spans the wavefront).
template <int MODE, int ROUNDS>
__device__ void ddrt_agg_body(const DDArgs& A) {
  using S = St<MODE>;
  const SortJob& s = *A.job;
  const uint32_t buf = s.npasses & 1;
  const unsigned long long* k = s.keys[buf];
  const uint32_t* v = s.vals[buf];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const uint32_t wid = blockIdx.x * (kT / 64) + w;
  const uint32_t wb = wid * (ROUNDS * 64);
  const uint32_t ns = dd_len(A);
  const bool packed = A.n < kPackLimit;
  uint32_t cf = 0, cb = 0;
  FS<MODE> fv = S::fid();
  BS<MODE> bv = S::bid();
  if (wb < ns) {  // (the sorted elements may be far fewer than the launch has room for)
#pragma unroll 1
    for (int r = ROUNDS - 1; r >= 0; --r) {
      uint8_t a;
      bool head, tail;
      load_round(k, v, A.aux, ns, packed, wb + r * 64 + lane, a, head, tail);
      uint32_t f = head;
      FS<MODE> x = S::flift(a);
      wave_fscan<MODE>(f, x);
      const uint32_t f63 = (uint32_t)__shfl((int)f, 63, 64);
      const FS<MODE> x63 = S::shfl(x, 63);
      fv = S::fop(x63, fv);  // this round, then the later ones
      if (f63) {
        cf = 1;
        break;
      }
    }
#pragma unroll 1
    for (int r = 0; r < ROUNDS; ++r) {
      uint8_t a;
      bool head, tail;
      load_round(k, v, A.aux, ns, packed, wb + r * 64 + lane, a, head, tail);
      uint32_t g = tail;
      BS<MODE> y = S::blift(a);
      wave_bscan<MODE>(g, y);
      const uint32_t g0 = (uint32_t)__shfl((int)g, 0, 64);
      const BS<MODE> y0 = S::shfl(y, 0);
      bv = S::bop(bv, y0);
      if (g0) {
        cb = 1;
        break;
      }
    }
  }
  if (lane == 0) {
    WaveAgg& o = A.agg[wid];
    o.ff = cf;
    o.bf = cb;
    put_f<MODE>(o.fs, fv);
    put_b<MODE>(o.bs, bv);
  }
}

template <int ROUNDS>
__global__ __launch_bounds__(kT) void ddrt_agg_kernel(DDArgs A) {
  if (A.ctl->max_ep < 4) ddrt_agg_body<0, ROUNDS>(A); else ddrt_agg_body<1, ROUNDS>(A);
}

// Carries between wavefronts (one block of 1,024 threads): the forward
// carry-in of wavefront i folds wavefronts < i, the backward carry-in folds
// wavefronts > i. Each thread folds a run of consecutive wavefronts; the runs'
// folds are scanned across the block (shuffles inside a wavefront, then the
// wavefront totals), and each thread walks its run again writing the carries.
// Forward element (ff, fs): a later element with ff set replaces the state.
// Backward element (bf, bs): an earlier element with bf set blocks what
// comes after it.
constexpr int kCT = 1024;

template <int MODE>
struct FwdEl {
  uint32_t f;
  FS<MODE> v;
};
template <int MODE>
struct BwdEl {
  uint32_t f;
  BS<MODE> v;
};

template <int MODE>
__device__ __forceinline__ FwdEl<MODE> fcomb(const FwdEl<MODE>& a, const FwdEl<MODE>& b) {  // a earlier
  return FwdEl<MODE>{a.f | b.f, b.f ? b.v : St<MODE>::fop(a.v, b.v)};
}
template <int MODE>
__device__ __forceinline__ BwdEl<MODE> bcomb(const BwdEl<MODE>& a, const BwdEl<MODE>& b) {  // a earlier
  return BwdEl<MODE>{a.f | b.f, a.f ? a.v : St<MODE>::bop(a.v, b.v)};
}

// The wavefront aggregates are split into kCT/64 contiguous ranges, one per
// wavefront, read in coalesced rounds of 64 and scanned with the segmented
// wavefront scans: a first sweep gives each wavefront's forward and backward
// totals, LDS carries them across wavefronts, and a second sweep writes every
// element's exclusive forward prefix and backward suffix.
// Each sweep loads the aggregates of its next round while it scans the
// current one (agg_raw), so its rounds wait on one load each in turn.
__device__ __forceinline__ WaveAgg agg_raw(const DDArgs& A, uint32_t e, uint32_t end) {
  WaveAgg g{};
  if (e < end) g = A.agg[e];
  return g;
}
template <int MODE>
__device__ __forceinline__ void load_agg(const WaveAgg& g, uint32_t e, uint32_t end, FwdEl<MODE>& x, BwdEl<MODE>& y) {
  using S = St<MODE>;
  if (e < end) {
    x = FwdEl<MODE>{g.ff, get_f<MODE>(g.fs)};
    y = BwdEl<MODE>{g.bf, get_b<MODE>(g.bs)};
  } else {
    x = FwdEl<MODE>{0, S::fid()};
    y = BwdEl<MODE>{0, S::bid()};
  }
}

template <int MODE>
__device__ void ddrt_carry_body(const DDArgs& A, uint32_t nw) {
  using S = St<MODE>;
  constexpr int kW = kCT / 64;
  __shared__ FwdEl<MODE> wf[kW];
  __shared__ BwdEl<MODE> wbk[kW];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const uint32_t rounds = ceil_div32(nw, kCT);
  const uint32_t c0 = min(nw, (uint32_t)w * rounds * 64), c1 = min(nw, c0 + rounds * 64);
  // sweep 1: this wavefront's totals
  FwdEl<MODE> tf{0, S::fid()};
  BwdEl<MODE> tb{0, S::bid()};
  WaveAgg g = agg_raw(A, c0 + lane, c1), gn{};
  for (uint32_t r = 0; r < rounds; ++r) {
    if (r + 1 < rounds) gn = agg_raw(A, c0 + (r + 1) * 64 + lane, c1);
    FwdEl<MODE> x;
    BwdEl<MODE> y;
    load_agg<MODE>(g, c0 + r * 64 + lane, c1, x, y);
    g = gn;
    wave_fscan<MODE>(x.f, x.v);
    wave_bscan<MODE>(y.f, y.v);
    tf = fcomb<MODE>(tf, FwdEl<MODE>{lane32(x.f, 63), S::lane(x.v, 63)});
    tb = bcomb<MODE>(tb, BwdEl<MODE>{lane32(y.f, 0), S::lane(y.v, 0)});  // rounds in order: earlier first
  }
  if (lane == 0) {
    wf[w] = tf;
    wbk[w] = tb;
  }
  __syncthreads();
  FwdEl<MODE> run{0, S::fid()};
  for (int q = 0; q < w; ++q) run = fcomb<MODE>(run, wf[q]);
  BwdEl<MODE> runb{0, S::bid()};
  for (int q = kW - 1; q > w; --q) runb = bcomb<MODE>(wbk[q], runb);
  // sweep 2: exclusive prefixes (forward, in order) and suffixes (backward)
  g = agg_raw(A, c0 + lane, c1);
  for (uint32_t r = 0; r < rounds; ++r) {
    const uint32_t e = c0 + r * 64 + lane;
    if (r + 1 < rounds) gn = agg_raw(A, e + 64, c1);
    FwdEl<MODE> x;
    BwdEl<MODE> y;
    load_agg<MODE>(g, e, c1, x, y);
    g = gn;
    wave_fscan<MODE>(x.f, x.v);
    const FwdEl<MODE> xp{dpp32<kDppWaveShr1>(0u, x.f), S::template dpp<kDppWaveShr1>(S::fid(), x.v)};
    const FwdEl<MODE> ex = lane == 0 ? run : fcomb<MODE>(run, xp);
    if (e < c1) put_f<MODE>(A.carry[e].fs, ex.v);
    run = fcomb<MODE>(run, FwdEl<MODE>{lane32(x.f, 63), S::lane(x.v, 63)});
  }
  if (rounds) g = agg_raw(A, c0 + (rounds - 1) * 64 + lane, c1);
  for (uint32_t r = rounds; r-- > 0;) {
    const uint32_t e = c0 + r * 64 + lane;
    if (r > 0) gn = agg_raw(A, e - 64, c1);
    FwdEl<MODE> x;
    BwdEl<MODE> y;
    load_agg<MODE>(g, e, c1, x, y);
    g = gn;
    wave_bscan<MODE>(y.f, y.v);
    const BwdEl<MODE> yn{dpp32<kDppWaveShl1>(0u, y.f), S::template dpp<kDppWaveShl1>(S::bid(), y.v)};
    const BwdEl<MODE> ex = lane == 63 ? runb : bcomb<MODE>(yn, runb);
    if (e < c1) put_b<MODE>(A.carry[e].bs, ex.v);
    runb = bcomb<MODE>(BwdEl<MODE>{lane32(y.f, 0), S::lane(y.v, 0)}, runb);
  }
}

__global__ __launch_bounds__(kCT) void ddrt_carry_kernel(DDArgs A, uint32_t nw) {
  nw = min(nw, ceil_div32(dd_len(A), kWaveElems));  // wavefronts that hold sorted elements
  if (A.ctl->max_ep < 4) ddrt_carry_body<0>(A, nw); else ddrt_carry_body<1>(A, nw);
}

// ROUNDS: rounds of 64 elements per wavefront. MID: the carries come from the
// wavefronts' aggregates themselves, 64 at a time back to the latest group
// start (and on to the next group end) instead of from the carry kernel, and
// the unused-transfer results are merged here (A.uth).
template <int MODE, int ROUNDS, bool MID>
__device__ void ddrt_final_body(const DDArgs& A, uint32_t (*s_val)[ROUNDS * 64], uint8_t (*s_code)[ROUNDS * 64]) {
  using S = St<MODE>;
  const SortJob& s = *A.job;
  const uint32_t buf = s.npasses & 1;
  const unsigned long long* k = s.keys[buf];
  const uint32_t* v = s.vals[buf];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const uint32_t wid = blockIdx.x * (kT / 64) + w;
  const uint32_t wb = wid * (ROUNDS * 64);
  // per round: value and endpoint code (LDS), start/end flags and forward results (bits)
  uint32_t heads, tails, fres = 0;
  const uint32_t ns = dd_len(A);
  if (blockIdx.x * (uint32_t)(kT * ROUNDS) >= ns) {  // past the sorted elements
    if (threadIdx.x == 0) {
      for (uint32_t k = S_DD_EVENTS; k <= S_ELIM_TX; ++k) *A.parts.at(k) = 0;
      if (MID)
        for (uint32_t k = S_UT_EVENTS; k <= S_UT_TIME; ++k) *A.parts.at(k) = 0;
    }
    return;
  }
  uint32_t unread;  // bit r: this lane's element of round r is an unused transfer
  load_wave<ROUNDS>(k, v, A.aux, ns, A.n < kPackLimit, wb, s_val[w], s_code[w], heads, tails, unread);
  // (what the classification found counts in a chronological log)
  if (!MID && A.ctl->first_bad != kNone) unread = 0;
  FS<MODE> carry = S::fid();
  BS<MODE> bcarry = S::bid();
  if constexpr (MID) {
    for (int r = 0; r < ROUNDS; ++r)
      if (wb + r * 64 + lane < ns) unread |= (uint32_t)A.uth[s_val[w][r * 64 + lane]] << r;
    for (int e = (int)wid - 1; e >= 0; e -= 64) {
      const int q = e - 63 + lane;
      uint32_t f = 0;
      FS<MODE> x = S::fid();
      if (q >= 0) {
        f = A.agg[q].ff;
        x = get_f<MODE>(A.agg[q].fs);
      }
      wave_fscan<MODE>(f, x);
      carry = S::fop(S::lane(x, 63), carry);
      if (lane32(f, 63)) break;
    }
    const int nw = (int)(gridDim.x * (kT / 64));
    for (int e = (int)wid + 1; e < nw; e += 64) {
      const int q = e + lane;
      uint32_t g = 0;
      BS<MODE> y = S::bid();
      if (q < nw) {
        g = A.agg[q].bf;
        y = get_b<MODE>(A.agg[q].bs);
      }
      wave_bscan<MODE>(g, y);
      bcarry = S::bop(bcarry, S::lane(y, 0));
      if (lane32(g, 0)) break;
    }
  } else {
    carry = get_f<MODE>(A.carry[wid].fs);
    bcarry = get_b<MODE>(A.carry[wid].bs);
  }
#pragma unroll 1
  for (int r = 0; r < ROUNDS; ++r) {
    const uint8_t a = s_code[w][r * 64 + lane];
    const bool head = (heads >> r) & 1;
    uint32_t f = head;
    FS<MODE> x = S::flift(a);
    wave_fscan<MODE>(f, x);
    // exclusive state of this lane
    const uint32_t fp = (uint32_t)__shfl_up((int)f, 1, 64);
    const FS<MODE> xp = S::shfl_up(x, 1);
    FS<MODE> ex = lane == 0 ? carry : (fp ? xp : S::fop(carry, xp));
    if (head) ex = S::fid();
    if (a != kNotTransfer) {
      const uint32_t sr = a >> 4, d = a & 15;
      if (S::has_dst(ex, d)) fres |= 1u << (2 * r);
      if (sr != d && S::rx(ex, sr, d)) fres |= 2u << (2 * r);
    }
    const uint32_t f63 = (uint32_t)__shfl((int)f, 63, 64);
    const FS<MODE> x63 = S::shfl(x, 63);
    carry = f63 ? x63 : S::fop(carry, x63);
  }
  unsigned long long c_ut = 0, b_ut = 0, t_ut = 0;
  unsigned long long c_dd = 0, c_grp = 0, c_tx = 0, c_rx = 0, b_dd = 0, t_dd = 0, b_rx = 0, t_rx = 0, t_el = 0;
#pragma unroll 1
  for (int r = ROUNDS - 1; r >= 0; --r) {
    const uint32_t j = wb + r * 64 + lane;
    const uint8_t a = s_code[w][r * 64 + lane];
    const bool tail = (tails >> r) & 1;
    uint32_t g = tail;
    BS<MODE> y = S::blift(a);
    wave_bscan<MODE>(g, y);
    const uint32_t gn = (uint32_t)__shfl_down((int)g, 1, 64);
    const BS<MODE> yn = S::shfl_down(y, 1);
    BS<MODE> ex = lane == 63 ? bcarry : (gn ? yn : S::bop(yn, bcarry));
    if (tail) ex = S::bid();
    if (j < ns && a != kNotTransfer) {
      const uint32_t sr = a >> 4, d = a & 15;
      uint8_t res = 0;
      if (fres & (1u << (2 * r))) res |= ODP_F_DD;
      if (fres & (2u << (2 * r))) res |= ODP_F_RT_RX;
      if (sr != d && S::tx(ex, sr, d)) res |= ODP_F_RT_TX;
      const bool found = res != 0;
      if ((unread >> r) & 1) res |= ODP_F_UT;
      c_grp += !(res & ODP_F_DD) && S::has_dst(ex, d);
      c_dd += (res & ODP_F_DD) != 0;
      c_tx += (res & ODP_F_RT_TX) != 0;
      c_rx += (res & ODP_F_RT_RX) != 0;
      // the classification stored the other records' flags (MID: 0 for every valid record)
      if (MID ? res != 0 : found) A.flags[s_val[w][r * 64 + lane]] = res;
      s_code[w][r * 64 + lane] = res;  // the code is not read again
    } else {
      s_code[w][r * 64 + lane] = 0;
    }
    const uint32_t g0 = (uint32_t)__shfl((int)g, 0, 64);
    const BS<MODE> y0 = S::shfl(y, 0);
    bcarry = g0 ? y0 : S::bop(y0, bcarry);
  }
  // bytes and durations of the flagged records, four rounds of gathers in flight at a time
  constexpr int kG = ROUNDS < 4 ? ROUNDS : 4;
  wave_lds_fence();
#pragma unroll 1
  for (int r0 = 0; r0 < ROUNDS; r0 += kG) {
    uint64_t eb[kG], ed[kG];
    uint8_t rs[kG];
#pragma unroll
    for (int q = 0; q < kG; ++q) {
      rs[q] = s_code[w][(r0 + q) * 64 + lane];
      eb[q] = ed[q] = 0;
      if (rs[q] & (ODP_F_DD | ODP_F_RT_RX | (MID ? ODP_F_UT : 0))) {
        const odp_event& e = A.ev[s_val[w][(r0 + q) * 64 + lane]];
        eb[q] = e.bytes;
        ed[q] = e.t_end - e.t_start;
      }
    }
#pragma unroll
    for (int q = 0; q < kG; ++q) {
      if (MID || !(rs[q] & ODP_F_UT)) t_el += ed[q];  // removable once, whether DD, RT_RX or both (UT: counted with those)
      if (rs[q] & ODP_F_DD) {
        b_dd += eb[q];
        t_dd += ed[q];
      }
      if (rs[q] & ODP_F_RT_RX) {
        b_rx += eb[q];
        t_rx += ed[q];
      }
      if (MID && (rs[q] & ODP_F_UT)) {
        ++c_ut;
        b_ut += eb[q];
        t_ut += ed[q];
      }
    }
  }
  block_store<R_ADD>(A.parts.at(S_DD_EVENTS), c_dd);
  block_store<R_ADD>(A.parts.at(S_DD_GROUPS), c_grp);
  block_store<R_ADD>(A.parts.at(S_DD_BYTES), b_dd);
  block_store<R_ADD>(A.parts.at(S_DD_TIME), t_dd);
  block_store<R_ADD>(A.parts.at(S_RT_PAIRS), c_tx);
  block_store<R_ADD>(A.parts.at(S_RT_RX), c_rx);
  block_store<R_ADD>(A.parts.at(S_RT_BYTES), b_rx);
  block_store<R_ADD>(A.parts.at(S_RT_TIME), t_rx);
  block_store<R_ADD>(A.parts.at(S_ELIM_TX), t_el);
  if constexpr (MID) {
    block_store<R_ADD>(A.parts.at(S_UT_EVENTS), c_ut);
    block_store<R_ADD>(A.parts.at(S_UT_BYTES), b_ut);
    block_store<R_ADD>(A.parts.at(S_UT_TIME), t_ut);
  }
}

template <int ROUNDS, bool MID>
__global__ __launch_bounds__(kT) void ddrt_final_kernel(DDArgs A) {
  __shared__ uint32_t s_val[kT / 64][ROUNDS * 64];
  __shared__ uint8_t s_code[kT / 64][ROUNDS * 64];
  if (A.ctl->max_ep < 4) ddrt_final_body<0, ROUNDS, MID>(A, s_val, s_code);
  else ddrt_final_body<1, ROUNDS, MID>(A, s_val, s_code);
}

// ---------------------------------------------------------------------------
// 5. Allocation/deletion pairing and the paired-allocation list.
// ---------------------------------------------------------------------------
struct PairArgs {
  const odp_event* ev;
  const SortJob* ad_job;
  const uint32_t* n_ad;
  const uint32_t* ad_idx;
  const uint8_t* ad_op;
  const uint64_t* ad_w_dev;
  const uint64_t* ad_w_addr;
  uint32_t* ad_alloc_partner;
  uint32_t* tile_cnt;
  // pair list
  uint32_t* pr_alloc;  // AD positions
  uint32_t* pr_del;
  uint64_t* pr_w_bytes;
  uint64_t* pr_w_dev;
  uint64_t* pr_w_haddr;
  uint8_t* flags;
  AnaCtl* ctl;
  odp_report* rep;
};

__global__ __launch_bounds__(kT) void pair_kernel(PairArgs P) {
  const uint32_t n = *P.n_ad;
  const SortJob& s = *P.ad_job;
  const uint32_t* v = s.vals[s.npasses & 1];
  for (uint32_t j = blockIdx.x * kT + threadIdx.x; j < n; j += gridDim.x * kT) {
    if (j == 0) continue;
    const uint32_t p = v[j], q = v[j - 1];
    if (P.ad_op[p] == ODP_DELETE && P.ad_op[q] == ODP_ALLOC && P.ad_w_dev[p] == P.ad_w_dev[q] &&
        P.ad_w_addr[p] == P.ad_w_addr[q])
      P.ad_alloc_partner[q] = p;
  }
}

__global__ __launch_bounds__(kT) void pair_count_kernel(PairArgs P) {
  const uint32_t n = *P.n_ad;
  const uint32_t b = blockIdx.x * kTile;
  if (b >= n) {
    if (threadIdx.x == 0) P.tile_cnt[2 * blockIdx.x] = P.tile_cnt[2 * blockIdx.x + 1] = 0;
    return;
  }
  uint32_t c = 0;
  for (uint32_t x = threadIdx.x; x < (uint32_t)kTile; x += kT) {
    const uint32_t p = b + x;
    if (p < n) c += P.ad_alloc_partner[p] != kNone;
  }
  for (int o = 32; o >= 1; o >>= 1) c += __shfl_xor(c, o, 64);
  __shared__ uint32_t sh[kT / 64];
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t t = 0;
    for (int w = 0; w < kT / 64; ++w) t += sh[w];
    P.tile_cnt[2 * blockIdx.x] = t;
    P.tile_cnt[2 * blockIdx.x + 1] = 0;
  }
}

__global__ __launch_bounds__(kT) void pair_scatter_kernel(PairArgs P) {
  const uint32_t n = *P.n_ad;
  const uint32_t b = blockIdx.x * kTile;
  if (b >= n) return;
  __shared__ uint32_t wc[kT / 64];
  __shared__ uint32_t run;
  if (threadIdx.x == 0) run = P.tile_cnt[2 * blockIdx.x];
  __syncthreads();
  const int w = threadIdx.x >> 6;
  unsigned long long unp_a = 0;
  for (uint32_t r = 0; r < (uint32_t)kItems; ++r) {
    const uint32_t p = b + r * kT + threadIdx.x;
    const bool in = p < n;
    const uint32_t partner = in ? P.ad_alloc_partner[p] : kNone;
    const bool paired_alloc = partner != kNone;
    const uint64_t m = __ballot(paired_alloc);
    if ((threadIdx.x & 63) == 0) wc[w] = __popcll(m);
    __syncthreads();
    uint32_t k = run;
    for (int x = 0; x < w; ++x) k += wc[x];
    k += __popcll(m & lanemask_lt());
    if (paired_alloc) {
      const odp_event& e = P.ev[P.ad_idx[p]];
      const uint64_t dv = P.ad_w_dev[p];
      P.pr_alloc[k] = p;
      P.pr_del[k] = partner;
      P.pr_w_bytes[k] = e.bytes;
      P.pr_w_dev[k] = dv;
      P.pr_w_haddr[k] = e.src_addr;
      P.flags[P.ad_idx[partner]] = ODP_F_PAIRED;  // the DELETE of the pair
    } else if (in && P.ad_op[p] == ODP_ALLOC) {
      ++unp_a;
    }
    __syncthreads();
    if (threadIdx.x == 0)
      for (int x = 0; x < kT / 64; ++x) run += wc[x];
    __syncthreads();
  }
  block_add(&P.rep->n_unpaired_alloc, unp_a);
}

// ---------------------------------------------------------------------------
// 6. Kernel lists per device (sorted by device, then start / end).
// ---------------------------------------------------------------------------
// Also writes the two sorted orders out as plain arrays of starts and ends,
// so the binary searches of the unused-mapping rules read one array each.
struct KernRangeArgs {
  const SortJob *ks, *ke;
  const uint64_t *k_w_dev, *k_w_start, *k_w_end;
  const uint32_t* n_k;
  uint64_t *starts_sorted, *ends_sorted;
  AnaCtl* ctl;
};
// (grid-stride; run by side_misc_kernel)
__device__ __forceinline__ void kernel_ranges_body(const KernRangeArgs& K) {
  const SortJob* ks = K.ks;
  const SortJob* ke = K.ke;
  const uint64_t* k_w_dev = K.k_w_dev;
  const uint64_t* k_w_start = K.k_w_start;
  const uint64_t* k_w_end = K.k_w_end;
  uint64_t* starts_sorted = K.starts_sorted;
  uint64_t* ends_sorted = K.ends_sorted;
  AnaCtl* ctl = K.ctl;
  const uint32_t* n_k = K.n_k;
  if (!ctl->kern_sort) return;  // the chronological path reads the per-device lists instead
  const uint32_t n = *n_k;
  const uint32_t* v = ks->vals[ks->npasses & 1];
  const uint32_t* ve = ke->vals[ke->npasses & 1];
  for (uint32_t j = blockIdx.x * kT + threadIdx.x; j < n; j += gridDim.x * kT) {
    const uint32_t d = (uint32_t)k_w_dev[v[j]];
    if (j == 0 || (uint32_t)k_w_dev[v[j - 1]] != d) ctl->dev_lo[d] = j;
    if (j + 1 == n || (uint32_t)k_w_dev[v[j + 1]] != d) ctl->dev_hi[d] = j + 1;
    starts_sorted[j] = k_w_start[v[j]];
    ends_sorted[j] = k_w_end[ve[j]];
  }
}

// ---------------------------------------------------------------------------
// 7. Repeated and unused allocations, flags of paired allocations.
// ---------------------------------------------------------------------------
// Groups of paired allocations by (host address, device, bytes) (Def. 3,
// Alg. 3's key) in an open-addressing table instead of a sort: RA needs, per
// pair, only whether an earlier pair of its key exists, and the rule's groups.
// Each pair probes linearly from the hash of its key and either claims an
// empty slot (its owner word, by compare-and-swap) or joins the slot whose
// owner has the same key, comparing the three key words of the owner, which
// the pair list already holds, so no thread waits for another. A slot keeps
// the smallest pair index of its key (pairs are numbered in ALLOC log order,
// so that is the first ALLOC) and whether a second pair joined it. Keys of
// many pairs are the common case (one hot buffer re-mapped again and again),
// so the owner and the smallest index are read first and written atomically
// only when that can change them, and "joined" is a plain store of 1. The
// table has a power of two >= 2 x (pairs) slots, so a probe always ends.
struct PairTable {
  uint32_t* owner;  // 0 empty, else 1 + the pair that claimed the slot
  uint32_t* first;  // smallest pair index of the slot's key
  uint32_t* multi;  // 1 when two or more pairs have the slot's key
  uint32_t* slot;   // per pair: the slot of its key
};

__host__ __device__ __forceinline__ uint32_t pair_table_mask(uint32_t n_pairs) {
  uint64_t c = 1024;
  while (c < 2ull * n_pairs) c <<= 1;
  return (uint32_t)(c - 1);
}

__device__ __forceinline__ uint32_t pair_hash(uint64_t haddr, uint64_t dev, uint64_t bytes) {
  uint64_t h = haddr * 0x9E3779B97F4A7C15ull ^ (bytes + 0x632BE59BD9B4E019ull) ^ (dev << 57);
  h ^= h >> 31;
  h *= 0xBF58476D1CE4E5B9ull;
  h ^= h >> 29;
  return (uint32_t)h;
}

__device__ __forceinline__ bool same_pair_key(const uint64_t* haddr, const uint64_t* dev, const uint64_t* bytes,
                                              uint32_t a, uint32_t b) {
  return haddr[a] == haddr[b] && dev[a] == dev[b] && bytes[a] == bytes[b];
}

// (grid-stride; run by side_misc_kernel)
__device__ __forceinline__ void pair_table_clear_body(const PairTable& T, const uint32_t* n_pairs) {
  const uint32_t size = pair_table_mask(*n_pairs) + 1;
  for (uint32_t i = blockIdx.x * kT + threadIdx.x; i < size; i += gridDim.x * kT) {
    T.owner[i] = 0;
    T.first[i] = kNone;
    T.multi[i] = 0;
  }
}

__global__ __launch_bounds__(kT) void pair_table_insert_kernel(PairTable T, const uint32_t* n_pairs,
                                                              const uint64_t* haddr, const uint64_t* dev,
                                                              const uint64_t* bytes) {
  const uint32_t n = *n_pairs;
  const uint32_t tmask = pair_table_mask(n);
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t waves = gridDim.x * (kT / 64);
  for (uint32_t base = (blockIdx.x * (kT / 64) + (threadIdx.x >> 6)) * 64; base < n; base += waves * 64) {
    const uint32_t k = base + lane;
    const bool in = k < n;
    const uint64_t ha = in ? haddr[k] : 0, dv = in ? dev[k] : 0, by = in ? bytes[k] : 0;
    const uint32_t t0 = in ? pair_hash(ha, dv, by) & tmask : 0u;
    // Lanes of one key inside the wavefront: the lowest (the smallest pair
    // index) inserts for all of them. One round per distinct key, lane moves
    // only; every lane knows its leader afterwards.
    uint64_t pending = __ballot(in);
    uint32_t leader = lane;
    uint64_t group = 0;
    while (pending) {
      const int l = __builtin_ctzll(pending);
      const uint32_t lt0 = (uint32_t)__shfl((int)t0, l, 64);
      const uint64_t lha = __shfl(ha, l, 64), ldv = __shfl(dv, l, 64), lby = __shfl(by, l, 64);
      const bool same = ((pending >> lane) & 1) && t0 == lt0 && ha == lha && dv == ldv && by == lby;
      const uint64_t m = __ballot(same);
      pending &= ~m;
      if (same) leader = (uint32_t)l;
      if ((uint32_t)l == lane) group = m;
    }
    uint32_t t = t0;
    if (in && leader == lane) {
      // the probe loop's lanes leave at different trips: what they decide is
      // stored inside it, only the slot index leaves it
      const bool several = __popcll(group) > 1;
      for (uint32_t probe = 0; probe <= tmask; ++probe, t = (t + 1) & tmask) {
        // an owner once set never changes: a stale 0 only costs the CAS
        uint32_t o = T.owner[t];
        if (o == 0) o = atomicCAS(T.owner + t, 0u, k + 1);
        if (o == 0) {  // claimed
          if (several) T.multi[t] = 1;
          break;
        }
        if (same_pair_key(haddr, dev, bytes, o - 1, k)) {  // joined
          if (T.multi[t] == 0) T.multi[t] = 1;
          break;
        }
      }
      if (k < T.first[t]) atomicMin(T.first + t, k);
    }
    t = (uint32_t)__shfl((int)t, (int)leader, 64);
    if (in) T.slot[k] = t;
  }
}

struct RaArgs {
  const odp_event* ev;
  PairTable T;
  const uint64_t* starts_sorted;  // kernel starts in (device, start) order
  const uint64_t* ends_sorted;    // kernel ends in (device, end) order
  const uint32_t* n_pairs;
  const uint32_t* pr_alloc;
  const uint32_t* pr_del;
  const uint32_t* ad_idx;
  const uint64_t* pr_w_bytes;
  const uint64_t* pr_w_dev;
  const uint64_t* pr_w_haddr;
  const uint32_t* ad_kc;
  const uint64_t* ad_km;
  const uint64_t* kd_ts;
  AnaCtl* ctl;
  uint8_t* flags;
  Parts parts;  // one partial per block of each RA/UA sum
};


// Kernels on device code `dev` whose closed interval meets [lo, hi] (lo <= hi):
// those that start by hi, less those that end before lo (an interval that
// ends before lo also starts before hi). The two binary searches take the same
// steps, so their loads, a chain of some twenty each, are in flight together.
__device__ __forceinline__ uint32_t kernels_meeting(const uint64_t* starts, const uint64_t* ends, const AnaCtl* ctl,
                                                    uint32_t dev, uint64_t lo, uint64_t hi) {
  uint32_t s = ctl->dev_lo[dev], e = s, len = ctl->dev_hi[dev] - s;
  if (len == 0) return 0;
  for (; len > 1; len -= len / 2) {
    const uint32_t half = len / 2;
    const uint64_t x = starts[s + half - 1], y = ends[e + half - 1];
    s += x <= hi ? half : 0u;
    e += y < lo ? half : 0u;
  }
  s += starts[s] <= hi;
  e += ends[e] < lo;
  return s - e;
}

// UA in a chronological log, with K and M as for unused transfers: the pair is
// used when M(ALLOC) reaches the ALLOC's start, or a kernel is logged between
// the ALLOC and the DELETE (K(DELETE) > K(ALLOC)), or the first kernel logged
// after the DELETE starts by the DELETE's end. Otherwise the count form's two
// binary searches decide.
__global__ __launch_bounds__(kT) void ra_ua_kernel(RaArgs R) {
  const bool chrono = !R.ctl->kern_sort;
  const uint32_t n = *R.n_pairs;
  unsigned long long c_ra = 0, c_grp = 0, b_ra = 0, t_ra = 0, c_ua = 0, b_ua = 0, t_ua = 0, t_el = 0;
  for (uint32_t k = blockIdx.x * kT + threadIdx.x; k < n; k += gridDim.x * kT) {
    // the slot of k's key: its first pair (the earliest ALLOC), and whether it has more
    const uint32_t t = R.T.slot[k];
    const bool head = R.T.first[t] == k;
    const bool group2 = head && R.T.multi[t] != 0;
    const uint32_t ai = R.ad_idx[R.pr_alloc[k]], di = R.ad_idx[R.pr_del[k]];
    const odp_event& a = R.ev[ai];
    const odp_event& d = R.ev[di];
    const uint64_t dur = (a.t_end - a.t_start) + (d.t_end - d.t_start);
    uint8_t f = ODP_F_PAIRED;
    if (!head) {
      f |= ODP_F_RA;
      ++c_ra;
      b_ra += a.bytes;
      t_ra += dur;
    }
    c_grp += group2;
    const uint32_t dev = (uint32_t)R.pr_w_dev[k];
    bool used;
    if (chrono) {
      const uint32_t pa = R.pr_alloc[k], pd = R.pr_del[k];
      const uint32_t ka = R.ad_kc[pa], kd = R.ad_kc[pd], total = R.ctl->kd_total[dev];
      used = (ka > 0 && R.ad_km[pa] >= a.t_start) || kd != ka ||
             (kd < total && R.kd_ts[R.ctl->kd_base[dev] + kd] <= d.t_end);
    } else {
      used = kernels_meeting(R.starts_sorted, R.ends_sorted, R.ctl, dev, a.t_start, d.t_end) != 0;
    }
    if (!used) {
      f |= ODP_F_UA;
      ++c_ua;
      b_ua += a.bytes;
      t_ua += dur;
    }
    if (f & (ODP_F_RA | ODP_F_UA)) t_el += dur;  // the pair is removable once
    R.flags[ai] = f;
  }
  block_store<R_ADD>(R.parts.at(S_RA_EVENTS), c_ra);
  block_store<R_ADD>(R.parts.at(S_RA_GROUPS), c_grp);
  block_store<R_ADD>(R.parts.at(S_RA_BYTES), b_ra);
  block_store<R_ADD>(R.parts.at(S_RA_TIME), t_ra);
  block_store<R_ADD>(R.parts.at(S_UA_EVENTS), c_ua);
  block_store<R_ADD>(R.parts.at(S_UA_BYTES), b_ua);
  block_store<R_ADD>(R.parts.at(S_UA_TIME), t_ua);
  block_store<R_ADD>(R.parts.at(S_ELIM_PAIRS), t_el);
}

// ---------------------------------------------------------------------------
// 8. Unused transfers (Def. 4, transfer half; Alg. 5).
//
// A copy into device memory is unused when no kernel on that device can read
// it before the next copy to the same place (same receiving device, sending
// device and source address) begins, or ever when none follows: no kernel's
// closed interval meets [copy.t_start, next.t_start]. Over the copy-ins sorted
// stably by (endpoints, source address), the next copy of a record is the
// element after it when that has the same key. Results go to a byte per
// copy-in (its position in log order), merged into the flags after the join.
// ---------------------------------------------------------------------------
struct UtArgs {
  const odp_event* ev;
  uint32_t n;          // records
  const uint8_t* cls;
  WaveScan W;          // scanned
  const SortJob* ut_job;
  const uint32_t* n_ut;
  const uint32_t* ut_idx;
  const uint64_t* ut_w_addr;
  const uint64_t* ut_w_code;
  const uint64_t* ut_ts;
  const uint32_t* ut_kc;
  const uint64_t* ut_km;
  const uint64_t* starts_sorted;
  const uint64_t* ends_sorted;
  uint32_t* next_q;  // per copy-in (log order): the next copy of its place, or kNone
  uint8_t* ut_hit;   // per copy-in (log order): 1 unused, 0 used, 2 left to the sorted path
  const uint64_t* kd_ts;   // KERNEL records per device code in log order: start
  const uint32_t* kd_idx;  // ... and record index
  AnaCtl* ctl;
  uint8_t* flags;
  Parts parts;  // one partial per block of each UT sum
};

// In a chronological log (no record rejected), with K(c) the number of
// kernels on c's device logged before copy c, M(c) the latest end among them
// and k the first kernel on the device logged after c, whether a kernel meets
// [c.t_start, n.t_start] (n the next copy of c's place) is decided by:
//   M(c) >= c.t_start (K(c) > 0)   a kernel is still running: used
//   no k (K(c) counts them all)    nothing can read c later: unused
//   otherwise the next copy of c's place, searched forward among the copies
//   logged before k: if it starts before k does, c is overwritten unread
//   (unused); if it starts when k does, or there is none before k, k can
//   read c (used).
// Only the listed copies are searched and searched for (see the classification).
// The forward search stops after kUtWindow of them; a copy still undecided
// then, or any copy of a log with a rejected record, is left to the sorted
// path below, which the device then switches on.
// (512: with 8 devices a device's next kernel is often hundreds of copies away,
// and the sorted path costs more than the wider staging does: 2 million records
// 623 -> 495 us against a window of 64, one device unchanged.)
constexpr uint32_t kUtWindow = 512;

// What the forward search finds of copy-in q: 0 used, 1 unused, 2 undecided. The
// workgroup's copy-ins start at b0, one per thread, q = b0 + threadIdx.x; s_ix[x]
// and s_h[x] hold the record index (kNone past the last) and a hash of the place
// of copy-in b0 + 1 + x, for x < kT + WINDOW (s_h: and eight more words of
// anything); h is the hash of q's place. The copies before the device's next
// kernel are found by a binary search over the indices, then their hashes are
// compared eight at a time and equal ones in full; FAR of them when the kernel
// lies past the window.
template <uint32_t WINDOW, uint32_t FAR>
__device__ __forceinline__ uint8_t ut_decide(const UtArgs& U, const uint32_t* s_ix, const uint32_t* s_h, uint32_t b0, uint32_t q,
                                             uint32_t h) {
  const uint64_t code = U.ut_w_code[q], ts = U.ut_ts[q];
  const uint32_t d = (uint32_t)(code & 15), k = U.ut_kc[q], total = U.ctl->kd_total[d];
  if (k > 0 && U.ut_km[q] >= ts) return 0;  // a kernel is still running
  if (k == total) return 1;                 // no kernel follows
  const uint32_t kp = U.ctl->kd_base[d] + k, kidx = U.kd_idx[kp];
  const uint64_t sk = U.kd_ts[kp], addr = U.ut_w_addr[q];
  // end: the staged copies logged before the kernel, WINDOW of them at most
  uint32_t x = threadIdx.x, end = x, top = x + WINDOW;
  while (end < top) {
    const uint32_t mid = (end + top) / 2;
    if (s_ix[mid] > kidx) top = mid; else end = mid + 1;
  }
  uint8_t hit = 0;
  if (end == threadIdx.x + WINDOW) {
    hit = 2;  // unless the next copy is among them
    end = threadIdx.x + FAR;
  }
  for (; x < end; x += 8) {
    uint32_t eq = 0;
#pragma unroll
    for (uint32_t u = 0; u < 8; ++u) eq |= (s_h[x + u] == h ? 1u : 0u) << u;
    if (end - x < 8) eq &= (1u << (end - x)) - 1;
    while (eq) {
      const uint32_t c = b0 + 1 + x + (uint32_t)__builtin_ctz(eq);
      if (U.ut_w_addr[c] == addr && U.ut_w_code[c] == code) {
        hit = U.ut_ts[c] < sk ? 1 : 0;  // the next copy of the place
        break;
      }
      eq &= eq - 1;
    }
    if (eq) break;
  }
  return hit;
}

// A block takes kT consecutive copy-ins (one per thread) and stages what its
// searches can reach (the next kT + kUtWindow) in LDS. Where a kernel is rarer
// than that most copies look through all they may before the sorted path takes
// them, hence the hashes, and half of the window only: 2 million records, a
// kernel every 5,000 and 3,000 places, 796 us with the places themselves staged
// and compared one after another (363 us of them in this kernel), 511 by hashes
// (75), 491 with half the window; 8 devices 490, 441 and 439.
constexpr uint32_t kUtStage = kT + kUtWindow;

__global__ __launch_bounds__(kT) void ut_scan_kernel(UtArgs U) {
  const uint32_t n = *U.n_ut;
  const bool chrono = U.ctl->first_bad == kNone;
  if (!chrono) {
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      U.ctl->kern_sort = 1;
      if (n) U.ctl->ut_need_sort = 1;
    }
    return;
  }
  __shared__ uint32_t s_ix[kUtStage], s_h[kUtStage + 8];
  for (uint32_t b0 = blockIdx.x * kT; b0 < n; b0 += gridDim.x * kT) {
    for (uint32_t x = threadIdx.x; x < kUtStage; x += kT) {
      const uint32_t r = b0 + 1 + x;
      s_ix[x] = r < n ? U.ut_idx[r] : kNone;
      s_h[x] = r < n ? near_hash(U.ut_w_addr[r], U.ut_w_code[r]) : 0u;
    }
    __syncthreads();
    const uint32_t q = b0 + threadIdx.x;
    if (q < n && U.ut_hit[q] != kUtSeen) {
      const uint8_t hit = ut_decide<kUtWindow, kUtWindow / 2>(U, s_ix, s_h, b0, q, near_hash(U.ut_w_addr[q], U.ut_w_code[q]));
      U.ut_hit[q] = hit;
      if (hit == 2) {  // the sorted path takes it
        U.ctl->ut_need_sort = 1;
        U.ctl->kern_sort = 1;
      }
    }
    __syncthreads();
  }
}

// The sorted path (only when switched on). Over the copy-ins sorted stably by
// (endpoints, source address): the next copy of a copy's place is the element
// after it when that has the same key.
// A wavefront takes 64 consecutive sorted elements, so each lane gets its
// neighbour's key by a lane move and only the last lane loads one more.
// (grid-stride by wavefronts; run by side_misc_kernel)
__device__ __forceinline__ void ut_next_body(const UtArgs& U) {
  if (!U.ctl->ut_need_sort) return;
  const uint32_t n = *U.n_ut;
  const SortJob& s = *U.ut_job;
  const uint32_t* v = s.vals[s.npasses & 1];
  const int lane = threadIdx.x & 63;
  for (uint32_t j0 = blockIdx.x * kT + (threadIdx.x & ~63u); j0 < n; j0 += gridDim.x * kT) {
    const uint32_t j = j0 + lane;
    const bool in = j < n;
    const uint32_t q = in ? v[j] : 0u;
    const uint64_t a = in ? U.ut_w_addr[q] : 0ull, c = in ? U.ut_w_code[q] : 0ull;
    uint64_t an = __shfl_down(a, 1, 64), cn = __shfl_down(c, 1, 64);
    uint32_t qn = (uint32_t)__shfl_down((int)q, 1, 64);
    if (lane == 63 && j + 1 < n) {
      qn = v[j + 1];
      an = U.ut_w_addr[qn];
      cn = U.ut_w_code[qn];
    }
    if (in) U.next_q[q] = (j + 1 < n && an == a && cn == c) ? qn : kNone;
  }
}

// Three independent grid-stride jobs of the allocation path in one launch
// (each a launch of its own before, mostly returning at once): the kernel
// lists' ranges and sorted starts and ends, the next copy of each copy-in's
// place (both only on their sorted paths), and the clearing of the RA table.
__global__ __launch_bounds__(kT) void side_misc_kernel(KernRangeArgs K, UtArgs U, PairTable T, const uint32_t* n_pairs) {
  kernel_ranges_body(K);
  ut_next_body(U);
  pair_table_clear_body(T, n_pairs);
}

// Over the copy-ins in log order: whether a kernel on the receiving device
// meets [copy start, next copy start] (no upper end without a next copy). In a chronological log (no record rejected) a device's kernels
// in start order are in log order, and with K(q) the number of them logged
// before copy q and M(q) the latest end among those, a kernel meets the window
// of copy c with next copy n exactly when: M(c) reaches c's start (K(c) > 0),
// or a kernel is logged between c and n (K(n) > K(c)), or the first kernel
// logged after n starts at n's start (a tie). Without a next copy: M(c)
// reaches c's start, or any kernel is logged after c. Otherwise the two binary
// searches of the count form decide. The result goes to ut_hit (merged into
// the flags after the join); only copies the forward search left open are
// decided here in a chronological log.
__global__ __launch_bounds__(kT) void ut_eval_kernel(UtArgs U) {
  if (!U.ctl->ut_need_sort) return;
  const uint32_t n = *U.n_ut;
  const bool chrono = U.ctl->first_bad == kNone;
  for (uint32_t q = blockIdx.x * kT + threadIdx.x; q < n; q += gridDim.x * kT) {
    if (chrono && U.ut_hit[q] != 2) continue;
    const uint32_t dev = (uint32_t)(U.ut_w_code[q] & 15);
    const uint64_t ts = U.ut_ts[q];
    const uint32_t nq = U.next_q[q];
    bool read;
    if (chrono) {
      const uint32_t lo_d = U.ctl->dev_lo[dev], cnt = U.ctl->dev_hi[dev] - lo_d;
      const uint32_t k = U.ut_kc[q];
      read = k > 0 && U.ut_km[q] >= ts;
      if (!read) {
        if (nq != kNone) {
          const uint32_t kn = U.ut_kc[nq];
          read = kn != k || (kn < cnt && U.starts_sorted[lo_d + kn] == U.ut_ts[nq]);
        } else {
          read = k != cnt;
        }
      }
    } else {
      const uint64_t hi = nq != kNone ? U.ut_ts[nq] : ~0ull;
      read = kernels_meeting(U.starts_sorted, U.ends_sorted, U.ctl, dev, ts, hi) != 0;
    }
    U.ut_hit[q] = !read;
  }
}

// After the join, when the transfers' other flags are final.
// First the listed copy-ins: sets ODP_F_UT and adds up those their search
// found unused, and the removable time of those no other flag made removable
// (a record flagged DD or RT_RX too has its time counted there already). Four
// copy-ins per thread and step, their loads issued together: each is a chain
// of dependent loads (result, record index, then flag and record). In a log
// with a rejected record all copies are listed, and what the classification
// decided of them is overwritten.
// Then the kernels that the classification could not see: a copy it found
// unused is used if a kernel of an earlier wavefront on its device still runs
// at its start. A wavefront takes the 512 records of one of the
// classification's and reads on while records start before the latest of
// those ends (a copy flagged DD or RT_RX as well stays removable).
__global__ __launch_bounds__(kT) void ut_merge_kernel(UtArgs U) {
  constexpr uint32_t kU = 4;
  const uint32_t n = *U.n_ut;
  const uint32_t stride = gridDim.x * kT;
  const uint32_t n_bad = U.ctl->first_bad;
  const uint8_t stale = n_bad == kNone ? 0 : ODP_F_UT;
  unsigned long long c_ut = 0, b_ut = 0, t_ut = 0, t_el = 0;
  for (uint32_t q0 = blockIdx.x * kT + threadIdx.x; q0 < n; q0 += kU * stride) {
    bool hit[kU];
    uint32_t idx[kU];
#pragma unroll
    for (uint32_t u = 0; u < kU; ++u) {
      const uint32_t q = q0 + u * stride;
      hit[u] = q < n && U.ut_hit[q] == 1;
    }
#pragma unroll
    for (uint32_t u = 0; u < kU; ++u) idx[u] = hit[u] || (stale && q0 + u * stride < n) ? U.ut_idx[q0 + u * stride] : kNone;
    uint8_t f[kU];
    uint64_t ts[kU], te[kU], by[kU];
#pragma unroll
    for (uint32_t u = 0; u < kU; ++u) {
      f[u] = idx[u] != kNone ? U.flags[idx[u]] : 0;
      ts[u] = hit[u] ? U.ev[idx[u]].t_start : 0;
      te[u] = hit[u] ? U.ev[idx[u]].t_end : 0;
      by[u] = hit[u] ? U.ev[idx[u]].bytes : 0;
    }
#pragma unroll
    for (uint32_t u = 0; u < kU; ++u) {
      if (!hit[u]) {
        if (f[u] & stale) U.flags[idx[u]] = f[u] & ~stale;
        continue;
      }
      U.flags[idx[u]] = f[u] | ODP_F_UT;
      const uint64_t d = te[u] - ts[u];
      ++c_ut;
      b_ut += by[u];
      t_ut += d;
      if (!(f[u] & (ODP_F_DD | ODP_F_RT_RX))) t_el += d;
    }
  }
  const uint32_t lane = threadIdx.x & 63;
  if (!stale) {
    for (uint32_t wid = (blockIdx.x * kT + threadIdx.x) / 64; wid < U.W.nw; wid += stride / 64) {
      const uint32_t wb = wid * kSpanRecs;
      if (wb >= U.n) break;
      // the latest end of an earlier wavefront's kernel, per device code (lane)
      unsigned long long last = 0;
      uint32_t some = 0;
      if (lane < kEp) {
        const uint32_t chunk = wid / kScanChunk;
        last = max(U.W.kmax[(size_t)kEp * wid + lane], U.W.cmax[(size_t)kEp * chunk + lane]);
        some = (U.W.cnt[(size_t)kWaveCnt * wid + 3 + lane] + U.W.ccnt[(size_t)kWaveCnt * chunk + 3 + lane]) != 0;
      }
      if (!__ballot(some && last >= U.ev[wb].t_start)) continue;
      unsigned long long most = last;
      for (int o = 8; o >= 1; o >>= 1) most = max(most, __shfl_xor(most, o, 64));
      most = __shfl(most, 0, 64);
      for (uint32_t r = 0; r < (uint32_t)kSpan; ++r) {
        const uint32_t i = wb + r * 64 + lane;
        const bool in = i < U.n;
        const uint64_t ts = in ? U.ev[i].t_start : ~0ull;
        const bool mine = in && U.cls[i] >= C_SEEN;
        const uint8_t f = mine ? U.flags[i] : 0;
        const uint32_t d = f & ODP_F_UT ? (uint32_t)(U.ev[i].dst_dev + 1) : 0u;
        const unsigned long long end = __shfl(last, (int)d, 64);
        const uint32_t any = (uint32_t)__shfl((int)some, (int)d, 64);
        if ((f & ODP_F_UT) && any && end >= ts) {
          U.flags[i] = f & ~ODP_F_UT;
          const uint64_t dur = U.ev[i].t_end - ts;
          --c_ut;
          b_ut -= U.ev[i].bytes;
          t_ut -= dur;
          if (!(f & (ODP_F_DD | ODP_F_RT_RX))) t_el -= dur;
        }
        if (lane64(ts, 63) > most) break;
      }
    }
  }
  block_store<R_ADD>(U.parts.at(S_UT_EVENTS), c_ut);
  block_store<R_ADD>(U.parts.at(S_UT_BYTES), b_ut);
  block_store<R_ADD>(U.parts.at(S_UT_TIME), t_ut);
  block_store<R_ADD>(U.parts.at(S_ELIM_UT), t_el);
}

// The optimization-potential estimate (Sec. 7.6): the run's time is the span
// of the valid records; removing the flagged mappings would save elim_ns.
__device__ void write_estimate(odp_report* rep, bool any_valid, uint64_t t_min, uint64_t t_max, uint64_t elim) {
  const uint64_t span = any_valid ? t_max - t_min : 0;
  rep->span_ns = span;
  rep->elim_ns = elim;
  rep->predicted_speedup = span == 0 ? 1.0 : elim >= span ? (double)INFINITY : (double)span / (double)(span - elim);
}

// The last reduction (nb partials of the unused transfers' sums) and the rest of
// the report, in one block of kT threads.
__global__ __launch_bounds__(kT) void finalize_kernel(Parts parts, uint32_t nb, AnaCtl* ctl, odp_report* rep) {
  unsigned long long sum[4] = {};
  for (uint32_t b = threadIdx.x; b < nb; b += kT)
#pragma unroll
    for (uint32_t k = 0; k < 4; ++k) sum[k] += parts.p[(size_t)(S_UT_EVENTS + k) * parts.stride + b];
  __shared__ unsigned long long s_sum[4];
#pragma unroll
  for (uint32_t k = 0; k < 4; ++k) block_store<R_ADD>(&s_sum[k], sum[k]);
  if (threadIdx.x != 0) return;
  rep->n_alloc_pairs = ctl->n_pairs;
  rep->n_unpaired_delete = (ctl->n_ad - rep->n_unpaired_alloc - 2ull * ctl->n_pairs);
  rep->dd_members = rep->dd_events + rep->dd_groups;
  rep->ra_members = rep->ra_events + rep->ra_groups;
  rep->first_bad_event = ctl->first_bad;
  rep->status = ctl->first_bad != kNone ? 1 : 0;
  uint64_t ud_time = 0;  // what the classification decided counts in a chronological log
  rep->ut_events = s_sum[0];
  rep->ut_bytes = s_sum[1];
  rep->ut_time_ns = s_sum[2];
  if (rep->n_events && ctl->first_bad == kNone) {
    rep->ut_events += ctl->ud_events;
    rep->ut_bytes += ctl->ud_bytes;
    rep->ut_time_ns += ud_time = ctl->ud_time;
  }
  write_estimate(rep, rep->n_events > rep->n_invalid, ctl->t_min, ctl->t_max,
                 ctl->elim_tx + ctl->elim_pairs + s_sum[3] + ud_time);
}

// ---------------------------------------------------------------------------
// 9. Literal Algorithm 2 (comparison mode for three or more endpoints).
// ---------------------------------------------------------------------------
// Algorithm 2 keeps, for each digest h and endpoint d, the list R(h, d) of
// every valid transfer of h into d (over the whole log, in log order) and a
// count c(h, d); walking the transfers in log order, it records a transfer tx
// of h out of s with rx = R(h, s)[c(h, s)] when c(h, s) < |R(h, s)|, and then
// adds one to c(h, dst(tx)). So c(h, d) counts the recorded transfers into d
// so far, and rx can precede tx or come from a third endpoint.
// Within one digest's transfers in log order this is, equivalently: a transfer
// k out of s is recorded unless it is late for s (every transfer into s comes
// before k) and every transfer into s was recorded; the late ones decide in
// log order through one bit per endpoint, F(d) = some transfer into d is
// unrecorded, which only grows. A recorded k pairs with the m-th transfer into
// s, m = the recorded transfers into s before k.
// One wavefront per 64 sorted positions handles the digest groups that start
// there. Those that end there too are handled together, a lane per transfer:
// counts and ranks are bits of the lane's own group in ballots over all 64, and
// the late transfers of all groups decide side by side. A group that goes on
// past the 64 is read from its start, and handled in the same way if it fits
// into 64 lanes, else in three sweeps: counts per endpoint, then the decisions
// and its transfers listed by destination endpoint (in `lists`), then rx.
// Bound by the latency of these chains of dependent steps: 53 us for 200,000
// records of three devices when the groups of a wavefront were taken one after
// another, 20 us now.
struct Alg2Args {
  const SortJob* job;        // the digest job (keys/vals in buffer npasses & 1)
  const uint8_t* aux;
  uint32_t n;                // records of the log
  uint32_t* rx;              // [n] partner record, or kNone
  unsigned long long* npairs;
};

__global__ __launch_bounds__(kT) void alg2_fill_kernel(uint32_t* rx, uint32_t n, unsigned long long* npairs) {
  const uint32_t i = blockIdx.x * kT + threadIdx.x;
  if (i < n) rx[i] = kNone;
  if (i == 0) *npairs = 0;
}

// per-lane pick of arr[idx] (idx < kEp) from a wave-replicated array
__device__ __forceinline__ uint32_t pick(const uint32_t (&arr)[kEp], uint32_t idx) {
  uint32_t r = 0;
#pragma unroll
  for (int e = 0; e < kEp; ++e) r = (uint32_t)e == idx ? arr[e] : r;
  return r;
}
__device__ __forceinline__ uint64_t pick64(const uint64_t (&arr)[kEp], uint32_t idx) {
  uint64_t r = 0;
#pragma unroll
  for (int e = 0; e < kEp; ++e) r = (uint32_t)e == idx ? arr[e] : r;
  return r;
}

// endpoint codes (0 host, 1 + device) of a sorted position; a transfer when x
// (w: the value there)
__device__ __forceinline__ void alg2_codes(const Alg2Args& A, uint32_t w, bool& x, uint32_t& src, uint32_t& dst, uint32_t& rec) {
  const uint8_t a = unpack_ep(A.n < kPackLimit ? w >> 24 : A.aux[w]);
  rec = A.n < kPackLimit ? (w & kIdxMask) : w;
  x = a != kNotTransfer;
  src = x ? (uint32_t)(a >> 4) : 0u;
  dst = x ? (uint32_t)(a & 15) : 0u;
}

// The groups of a wavefront's 64 sorted positions from b on: G is the mask of the
// lanes of this lane's group, or 0 when the lane takes no part. Returns the
// number of transfers recorded. list: 64 words of LDS of the wavefront.
__device__ __forceinline__ uint32_t alg2_together(const Alg2Args& A, const uint32_t* v, uint32_t b, uint64_t G, uint32_t* list) {
  const uint32_t lane = threadIdx.x & 63;
  const uint64_t lt = lanemask_lt();
  bool x = false;
  uint32_t src = 0, dst = 0, rec = 0;
  if (G) alg2_codes(A, v[b + lane], x, src, dst, rec);
  uint64_t into[kEp];
#pragma unroll
  for (int e = 0; e < kEp; ++e) into[e] = __ballot(x && dst == (uint32_t)e);
  const uint64_t isrc = pick64(into, src) & G;
  const uint32_t before = (uint32_t)__popcll(isrc & lt);
  // every transfer into its source comes before it: late ones decide in log order
  uint32_t waits = x && before == (uint32_t)__popcll(isrc), u = 0, F = 0;
  for (;;) {
    const uint64_t c = __ballot(waits && !((F >> src) & 1)) & G;
    if (!__ballot(c != 0)) break;
    const uint32_t first = c ? (uint32_t)__builtin_ctzll(c) : lane;  // of this lane's group
    const uint32_t d = (uint32_t)__shfl((int)dst, (int)first, 64);
    F |= c ? 1u << d : 0u;
    u |= c && lane == first;
    waits = c && lane <= first ? 0u : waits;
  }
  uint64_t uinto[kEp];
  uint32_t at = G ? (uint32_t)__builtin_ctzll(G) : 0u, mine = 0, base_src = at;
#pragma unroll
  for (int e = 0; e < kEp; ++e) {
    uinto[e] = __ballot(u && dst == (uint32_t)e);
    if ((uint32_t)e == dst) mine = at;
    if ((uint32_t)e == src) base_src = at;
    at += (uint32_t)__popcll(into[e] & G);
  }
  if (x) list[mine + (uint32_t)__popcll(pick64(into, dst) & G & lt)] = rec;
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  const bool recorded = x && !u;
  const uint32_t m = before - (uint32_t)__popcll(pick64(uinto, src) & G & lt);
  if (recorded) A.rx[rec] = list[base_src + m];
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  return (uint32_t)__popcll(__ballot(recorded));
}

__global__ __launch_bounds__(kT) void alg2_kernel(Alg2Args A) {
  const SortJob& s = *A.job;
  const unsigned long long* k = s.keys[s.npasses & 1];
  const uint32_t* v = s.vals[s.npasses & 1];
  uint32_t* lists = s.vals[(s.npasses + 1) & 1];
  const uint32_t n = sorted_len(s), lane = threadIdx.x & 63;
  const uint64_t lt = lanemask_lt();
  const uint32_t c0 = (blockIdx.x * kT + threadIdx.x) / 64 * 64;
  if (c0 >= n) return;
  const uint32_t j = c0 + lane;
  const bool in = j < n;
  const unsigned long long key = in ? k[j] : 0ull;
  const bool head = in && (j == 0 || k[j - 1] != key);
  const bool tail = in && (j + 1 == n || k[j + 1] != key);
  __shared__ uint32_t s_list[kT / 64][64];
  uint32_t* list = s_list[threadIdx.x >> 6];
  const uint64_t heads = __ballot(head), tails = __ballot(tail), le = lt | 1ull << lane;
  const uint64_t starts = heads & le, ends = tails & ~lt;  // of this lane's group
  uint64_t G = 0;
  if (in && starts && ends) {
    const int from = 63 - __builtin_clzll(starts), to = __builtin_ctzll(ends);
    G = (to == 63 ? ~0ull : (1ull << (to + 1)) - 1) & ~((1ull << from) - 1);
  }
  uint64_t pairs = alg2_together(A, v, c0, G, list);
  // the group that starts here and goes on, if any
  const int last = heads ? 63 - __builtin_clzll(heads) : -1;
  if (last >= 0 && (tails >> last) == 0) {
    const uint32_t g0 = c0 + (uint32_t)last;
    const unsigned long long gkey = k[g0];
    const bool more = g0 + lane < n && k[g0 + lane] == gkey;
    const uint64_t members = __ballot(more);
    if (members != ~0ull || g0 + 64 >= n || k[g0 + 64] != gkey) {
      pairs += alg2_together(A, v, g0, more ? members : 0ull, list);
      if (lane == 0 && pairs) atomicAdd(A.npairs, (unsigned long long)pairs);
      return;
    }
    // (In each sweep the next 64 values are read before these are worked on: a
    // wavefront alone waits for every read. 300,000 records of one digest: 13.7 ms
    // without that, 12.8 so.)
    // sweep 1: transfers into each endpoint, and the group's end g1
    uint32_t cnt[kEp];
#pragma unroll
    for (int e = 0; e < kEp; ++e) cnt[e] = 0;
    uint32_t g1 = g0;
    uint32_t next = v[min(g0 + lane, n - 1)];
    unsigned long long knext = k[min(g0 + lane, n - 1)];
    for (uint32_t b = g0;; b += 64) {
      const uint32_t w = next;
      const bool inr = b + lane < n && knext == gkey;
      next = v[min(b + 64 + lane, n - 1)];
      knext = k[min(b + 64 + lane, n - 1)];
      bool x = false;
      uint32_t src = 0, dst = 0, rec = 0;
      if (inr) alg2_codes(A, w, x, src, dst, rec);
#pragma unroll
      for (int e = 0; e < kEp; ++e) cnt[e] += (uint32_t)__popcll(__ballot(x && dst == (uint32_t)e));
      const uint32_t m = (uint32_t)__popcll(__ballot(inr));
      g1 = b + m;
      if (m < 64) break;
    }
    uint32_t base[kEp];
    {
      uint32_t acc = g0;
#pragma unroll
      for (int e = 0; e < kEp; ++e) {
        base[e] = acc;
        acc += cnt[e];
      }
    }
    // sweep 2: decisions, each transfer's place in the list of its
    // destination, and the rank in R(h, src) of each recorded one (kept in
    // rx until sweep 3)
    uint32_t seen[kEp], unrec[kEp];
#pragma unroll
    for (int e = 0; e < kEp; ++e) seen[e] = unrec[e] = 0;
    uint32_t F = 0;
    next = v[min(g0 + lane, g1 - 1)];
    for (uint32_t b = g0; b < g1; b += 64) {
      const uint32_t w = next;
      next = v[min(b + 64 + lane, g1 - 1)];
      bool x = false;
      uint32_t src = 0, dst = 0, rec = 0;
      if (b + lane < g1) alg2_codes(A, w, x, src, dst, rec);
      uint64_t into[kEp];
#pragma unroll
      for (int e = 0; e < kEp; ++e) into[e] = __ballot(x && dst == (uint32_t)e);
      const uint32_t before_src = pick(seen, src) + (uint32_t)__popcll(pick64(into, src) & lt);
      const bool late = x && before_src == pick(cnt, src);
      uint64_t rest = __ballot(late), um = 0;
      while (rest) {
        const uint64_t c = __ballot(((rest >> lane) & 1) && !((F >> src) & 1));
        if (!c) break;
        const int k0 = __builtin_ctzll(c);
        um |= 1ull << k0;
        F |= 1u << __shfl((int)dst, k0, 64);
        rest &= k0 == 63 ? 0ull : ~0ull << (k0 + 1);
      }
      const bool u = (um >> lane) & 1;
      uint64_t uinto[kEp];
#pragma unroll
      for (int e = 0; e < kEp; ++e) uinto[e] = __ballot(u && dst == (uint32_t)e);
      if (x) {
        const uint32_t my_rank = pick(seen, dst) + (uint32_t)__popcll(pick64(into, dst) & lt);
        __hip_atomic_store(lists + pick(base, dst) + my_rank, rec, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint32_t m = before_src - pick(unrec, src) - (uint32_t)__popcll(pick64(uinto, src) & lt);
        __hip_atomic_store(A.rx + rec, u ? kNone : m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
#pragma unroll
      for (int e = 0; e < kEp; ++e) {
        seen[e] += (uint32_t)__popcll(into[e]);
        unrec[e] += (uint32_t)__popcll(uinto[e]);
      }
    }
    // the stores above reach the L2 before sweep 3 reads them past the L1
    __builtin_amdgcn_s_waitcnt(0);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    // sweep 3: rank -> record
    next = v[min(g0 + lane, g1 - 1)];
    for (uint32_t b = g0; b < g1; b += 64) {
      const uint32_t w = next;
      next = v[min(b + 64 + lane, g1 - 1)];
      bool x = false;
      uint32_t src = 0, dst = 0, rec = 0;
      if (b + lane < g1) alg2_codes(A, w, x, src, dst, rec);
      bool paired = false;
      if (x) {
        const uint32_t m = __hip_atomic_load(A.rx + rec, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (m != kNone) {
          paired = true;
          A.rx[rec] = __hip_atomic_load(lists + pick(base, src) + m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      }
      pairs += (uint64_t)__popcll(__ballot(paired));
    }
  }
  if (lane == 0 && pairs) atomicAdd(A.npairs, (unsigned long long)pairs);
}

#include "analyze_mid.h"

// ---------------------------------------------------------------------------
// Workspace layout.
// ---------------------------------------------------------------------------
enum Buf {
  B_CTL, B_JOBS, B_CLS, B_AUX, B_BKEY0, B_BKEY1, B_BVAL0, B_BVAL1, B_TILECNT, B_AD, B_K, B_PR, B_HIST,
  B_TOTALS, B_SEG, B_SKEY, B_PARTS, B_UT, B_WSCAN, B_MID
};

// Jobs 1..4 (the subsets) are sorted together in the same launches.
constexpr int kJobBig = 0, kJobAd = 1, kJobKs = 2, kJobKe = 3, kJobUt = 4, kNumJobs = 5;
constexpr int kSubsetJobs = 4;
static_assert(kTotals == kNumJobs * kMaxPasses * 256, "digit totals of every job");

template <typename T>
T* carve(char*& p, size_t count) {
  uintptr_t a = (reinterpret_cast<uintptr_t>(p) + 7) & ~uintptr_t(7);
  T* r = reinterpret_cast<T*>(a);
  p = reinterpret_cast<char*>(a + count * sizeof(T));
  return r;
}

// Every device array of the analysis, carved from the workspace buffers.
struct Views {
  size_t cap;
  uint32_t ntc;  // tiles of the capacity
  AnaCtl* ctl;
  SortJob* jobs;
  uint8_t* cls;
  uint8_t* aux;
  uint8_t* cand;
  unsigned long long* bk[2];
  uint32_t* bv[2];
  uint32_t* tile_cnt;
  uint32_t* wave_cnt;
  uint32_t* wave_copies;
  SubsetOut S;
  uint32_t* ad_vals1;
  uint32_t* k_vals_s1;
  uint32_t* k_vals_e1;
  uint64_t* starts_sorted;
  uint64_t* ends_sorted;
  uint32_t* ut_vals1;
  uint32_t* next_q;
  uint8_t* ut_hit;
  WaveScan wscan;
  uint32_t *pr_alloc, *pr_del;
  PairTable pt;
  uint64_t *pr_w_bytes, *pr_w_dev, *pr_w_haddr;
  uint32_t* hist;
  uint32_t* totals;
  WaveAgg* agg;    // per wavefront of the digest job
  WaveAgg* carry;
  unsigned long long* skey[2 * (kNumJobs - 1)];  // key ping-pong of the subset jobs
  Parts parts;                  // per-block partials of the grid-wide reductions
  MidView mid;
};

// Arrays of the analysis of up to kMidMax records, for a workspace of cap
// records; with base == null only their size is computed.
size_t mid_views(MidView& m, char* base, size_t cap) {
  const size_t c = (std::min<size_t>(cap, kMidMax) + kMidTile - 1) / kMidTile * kMidTile;
  const size_t slots = (size_t)pair_table_mask((uint32_t)c) + 1, waves = c / kClsWave, blocks = c / kClsT;
  char* p = base;
  m.gid0 = carve<uint32_t>(p, c);
  m.gid1 = carve<uint32_t>(p, c);
  p = reinterpret_cast<char*>((reinterpret_cast<uintptr_t>(p) + 15) & ~uintptr_t(15));
  m.dtab = carve<uint32_t>(p, slots);
  m.h0 = carve<uint32_t>(p, c / kMidTile * kMidDigits);
  m.h1 = carve<uint32_t>(p, c / kMidTile * kMidDigits);
  m.uth = carve<uint8_t>(p, c);
  m.ad_host = carve<uint64_t>(p, c);
  m.ad_bytes = carve<uint64_t>(p, c);
  m.kd_te = carve<uint64_t>(p, c);
  m.ks = carve<uint64_t>(p, c);
  m.ke = carve<uint64_t>(p, c);
  for (NearTable* t : {&m.ad, &m.ut}) {
    p = reinterpret_cast<char*>((reinterpret_cast<uintptr_t>(p) + 15) & ~uintptr_t(15));  // read four slots at once
    t->owner = carve<uint32_t>(p, slots);
    t->bits = carve<unsigned long long>(p, slots * kChunkWords);
    t->ckey = carve<uint32_t>(p, slots);
    t->clast = carve<uint32_t>(p, slots);
    t->link = carve<uint32_t>(p, c);
  }
  const size_t nchunk = waves / kScanChunk + 1;
  m.wscan.cnt = carve<uint32_t>(p, waves * kWaveCnt);
  m.wscan.kmax = carve<uint64_t>(p, waves * kEp);
  m.wscan.ccnt = carve<uint32_t>(p, nchunk * kWaveCnt);
  m.wscan.cmax = carve<uint64_t>(p, nchunk * kEp);
  m.wscan.nw = 0;
  m.wscan.copies = nullptr;
  m.agg = carve<WaveAgg>(p, waves);
  m.parts.p = carve<unsigned long long>(p, kSlots * blocks);
  m.parts.stride = (uint32_t)blocks;
  return (size_t)(p - base);
}

Views views(Workspace* ws) {
  Views v;
  DevBuf* b = ws->a_bufs;
  v.cap = ws->a_cap_events;
  v.ntc = ceil_div32(v.cap, kTile);
  v.ctl = static_cast<AnaCtl*>(b[B_CTL].ptr);
  v.jobs = static_cast<SortJob*>(b[B_JOBS].ptr);
  v.cls = static_cast<uint8_t*>(b[B_CLS].ptr);
  v.aux = static_cast<uint8_t*>(b[B_AUX].ptr);
  v.cand = v.aux + v.cap;
  v.bk[0] = static_cast<unsigned long long*>(b[B_BKEY0].ptr);
  v.bk[1] = static_cast<unsigned long long*>(b[B_BKEY1].ptr);
  v.bv[0] = static_cast<uint32_t*>(b[B_BVAL0].ptr);
  v.bv[1] = static_cast<uint32_t*>(b[B_BVAL1].ptr);
  v.tile_cnt = static_cast<uint32_t*>(b[B_TILECNT].ptr);
  v.wave_cnt = v.tile_cnt + 2 * (size_t)v.ntc;  // kWaveCnt counters per wavefront
  v.wave_copies = v.wave_cnt + (size_t)kWaveCnt * v.ntc * (kTile / kSpanRecs);  // one per wavefront
  const size_t cap = v.cap;
  char* pa = static_cast<char*>(b[B_AD].ptr);
  v.S.ad_idx = carve<uint32_t>(pa, cap);
  v.S.ad_w_dev = carve<uint64_t>(pa, cap);
  v.S.ad_w_addr = carve<uint64_t>(pa, cap);
  v.S.ad_vals = carve<uint32_t>(pa, cap);
  v.ad_vals1 = carve<uint32_t>(pa, cap);
  v.S.ad_alloc_partner = carve<uint32_t>(pa, cap);
  v.S.ad_kc = carve<uint32_t>(pa, cap);
  v.S.ad_km = carve<uint64_t>(pa, cap);
  v.S.ad_op = carve<uint8_t>(pa, cap);
  char* pk = static_cast<char*>(b[B_K].ptr);
  v.S.k_idx = carve<uint32_t>(pk, cap);
  v.S.k_w_start = carve<uint64_t>(pk, cap);
  v.S.k_w_end = carve<uint64_t>(pk, cap);
  v.S.k_w_dev = carve<uint64_t>(pk, cap);
  v.S.k_vals_s = carve<uint32_t>(pk, cap);
  v.k_vals_s1 = carve<uint32_t>(pk, cap);
  v.S.k_vals_e = carve<uint32_t>(pk, cap);
  v.k_vals_e1 = carve<uint32_t>(pk, cap);
  v.starts_sorted = carve<uint64_t>(pk, cap);
  v.ends_sorted = carve<uint64_t>(pk, cap);
  v.S.kd_ts = carve<uint64_t>(pk, cap);
  v.S.kd_idx = carve<uint32_t>(pk, cap);
  v.S.ctl = v.ctl;
  char* pu = static_cast<char*>(b[B_UT].ptr);
  v.S.ut_idx = carve<uint32_t>(pu, cap);
  v.S.ut_w_addr = carve<uint64_t>(pu, cap);
  v.S.ut_w_code = carve<uint64_t>(pu, cap);
  v.S.ut_ts = carve<uint64_t>(pu, cap);
  v.S.ut_vals = carve<uint32_t>(pu, cap);
  v.S.ut_kc = carve<uint32_t>(pu, cap);
  v.S.ut_km = carve<uint64_t>(pu, cap);
  v.ut_vals1 = carve<uint32_t>(pu, cap);
  v.next_q = carve<uint32_t>(pu, cap);
  v.ut_hit = carve<uint8_t>(pu, cap);
  v.S.ut_hit = v.ut_hit;
  char* pw = static_cast<char*>(b[B_WSCAN].ptr);
  const uint32_t nw = v.ntc * (kTile / kSpanRecs), nchunk = ceil_div32(nw, kScanChunk);
  v.wscan.cnt = v.wave_cnt;
  v.wscan.kmax = carve<uint64_t>(pw, (size_t)nw * kEp);
  v.wscan.ccnt = carve<uint32_t>(pw, (size_t)nchunk * kWaveCnt);
  v.wscan.cmax = carve<uint64_t>(pw, (size_t)nchunk * kEp);
  v.wscan.nw = nw;
  v.wscan.copies = nullptr;
  char* pp = static_cast<char*>(b[B_PR].ptr);
  v.pr_alloc = carve<uint32_t>(pp, cap);
  v.pr_del = carve<uint32_t>(pp, cap);
  v.pr_w_bytes = carve<uint64_t>(pp, cap);
  v.pr_w_dev = carve<uint64_t>(pp, cap);
  v.pr_w_haddr = carve<uint64_t>(pp, cap);
  const size_t tcap = (size_t)pair_table_mask((uint32_t)std::min<size_t>(cap / 2, 0x7FFFFFFFu)) + 1;
  v.pt.owner = carve<uint32_t>(pp, tcap);
  v.pt.first = carve<uint32_t>(pp, tcap);
  v.pt.multi = carve<uint32_t>(pp, tcap);
  v.pt.slot = carve<uint32_t>(pp, cap);
  v.hist = static_cast<uint32_t*>(b[B_HIST].ptr);
  v.totals = static_cast<uint32_t*>(b[B_TOTALS].ptr);
  char* ps = static_cast<char*>(b[B_SEG].ptr);
  v.agg = carve<WaveAgg>(ps, (size_t)v.ntc * (kT / 64));
  v.carry = carve<WaveAgg>(ps, (size_t)v.ntc * (kT / 64));
  char* pkey = static_cast<char*>(b[B_SKEY].ptr);
  for (int i = 0; i < 2 * (kNumJobs - 1); ++i) v.skey[i] = carve<unsigned long long>(pkey, cap);
  v.parts.p = static_cast<unsigned long long*>(b[B_PARTS].ptr);
  v.parts.stride = v.ntc;
  mid_views(v.mid, static_cast<char*>(b[B_MID].ptr), cap);
  return v;
}

// Sort job table for a workspace capacity (device-resident; the pass lists
// inside are refilled on the device by every call).
void build_jobs(const Views& v, SortJob* hj) {
  std::memset(static_cast<void*>(hj), 0, sizeof(SortJob) * kNumJobs);
  for (int j = 0; j < kNumJobs; ++j) hj[j].mono_word = kNoWord;
  AnaCtl* ctl = v.ctl;
  // all records by digest (keyed; non-transfers carry an all-ones key and contribute nothing)
  hj[kJobBig].n_ptr = &ctl->n;
  hj[kJobBig].keys[0] = v.bk[0];
  hj[kJobBig].keys[1] = v.bk[1];
  hj[kJobBig].vals[0] = v.bv[0];
  hj[kJobBig].vals[1] = v.bv[1];
  hj[kJobBig].masks[0] = &ctl->m_digest;
  hj[kJobBig].word_bytes[0] = 8;
  hj[kJobBig].nwords = 1;
  hj[kJobBig].hist0_pre = 1;
  hj[kJobBig].drop0 = 1;
  hj[kJobBig].n_after0 = &ctl->n_tx;
  hj[kJobBig].aux = v.aux;
  // ALLOC/DELETE by (device, device address); words least significant first
  hj[kJobAd].n_ptr = &ctl->n_ad;
  hj[kJobAd].vals[0] = v.S.ad_vals;
  hj[kJobAd].vals[1] = v.ad_vals1;
  hj[kJobAd].words[0] = v.S.ad_w_addr;
  hj[kJobAd].masks[0] = &ctl->m_ad_addr;
  hj[kJobAd].word_bytes[0] = 8;
  hj[kJobAd].words[1] = v.S.ad_w_dev;
  hj[kJobAd].masks[1] = &ctl->m_ad_dev;
  hj[kJobAd].word_bytes[1] = 1;
  hj[kJobAd].nwords = 2;
  // kernels by (device, start) and by (device, end)
  hj[kJobKs].n_ptr = &ctl->n_k;
  hj[kJobKs].vals[0] = v.S.k_vals_s;
  hj[kJobKs].vals[1] = v.k_vals_s1;
  hj[kJobKs].words[0] = v.S.k_w_start;
  hj[kJobKs].masks[0] = &ctl->m_k_start;
  hj[kJobKs].word_bytes[0] = 8;
  hj[kJobKs].words[1] = v.S.k_w_dev;
  hj[kJobKs].masks[1] = &ctl->m_k_dev;
  hj[kJobKs].word_bytes[1] = 1;
  hj[kJobKs].nwords = 2;
  hj[kJobKe] = hj[kJobKs];
  // Valid records are in non-decreasing t_start order when no record was
  // rejected (a rejected record can hide a decrease), so the kernels' starts
  // then need no sorting: a stable sort by device keeps them in order.
  hj[kJobKs].first_bad = &ctl->first_bad;
  hj[kJobKs].mono_word = 0;
  hj[kJobKs].run_flag = &ctl->kern_sort;
  hj[kJobKe].run_flag = &ctl->kern_sort;
  hj[kJobKe].vals[0] = v.S.k_vals_e;
  hj[kJobKe].vals[1] = v.k_vals_e1;
  hj[kJobKe].words[0] = v.S.k_w_end;
  hj[kJobKe].masks[0] = &ctl->m_k_end;
  // copy-ins by (endpoint code, source address): each group in log order
  hj[kJobUt].n_ptr = &ctl->n_ut;
  hj[kJobUt].vals[0] = v.S.ut_vals;
  hj[kJobUt].vals[1] = v.ut_vals1;
  hj[kJobUt].words[0] = v.S.ut_w_addr;
  hj[kJobUt].masks[0] = &ctl->m_ut_addr;
  hj[kJobUt].word_bytes[0] = 8;
  hj[kJobUt].words[1] = v.S.ut_w_code;
  hj[kJobUt].masks[1] = &ctl->m_ut_code;
  hj[kJobUt].word_bytes[1] = 1;
  hj[kJobUt].nwords = 2;
  hj[kJobUt].run_flag = &ctl->ut_need_sort;
  for (int j = 1; j < kNumJobs; ++j) {
    hj[j].keys[0] = v.skey[2 * (j - 1)];
    hj[j].keys[1] = v.skey[2 * (j - 1) + 1];
  }
  for (int j = 0; j < kNumJobs; ++j) {
    hj[j].ntiles_max = v.ntc;
    hj[j].hist = v.hist + (size_t)j * 256 * v.ntc;
    hj[j].totals = v.totals + (size_t)j * kMaxPasses * 256;
  }
}

}  // namespace

// A captured graph holds workspace addresses: dropped before anything moves.
static void analyze_drop_graph(Workspace* ws) {
  if (ws->a_graph) {
    (void)hipDeviceSynchronize();
    (void)hipGraphExecDestroy(ws->a_graph);
    ws->a_graph = nullptr;
  }
  ws->ag_ev = nullptr;
  ws->ag_n = 0;
}

int analyze_reserve(Workspace* ws, size_t max_events) {
  size_t cap = max_events < 4096 ? 4096 : max_events;
  if (cap <= ws->a_cap_events) return ODP_OK;
  analyze_drop_graph(ws);
  const uint32_t nt = ceil_div32(cap, kTile);
  DevBuf* b = ws->a_bufs;
  int e;
  MidView sized;
  if ((e = b[B_MID].ensure(mid_views(sized, nullptr, cap) + 64)) || (e = b[B_CTL].ensure(sizeof(AnaCtl))) || (e = b[B_JOBS].ensure(sizeof(SortJob) * kNumJobs)) ||
      (e = b[B_CLS].ensure(cap)) || (e = b[B_AUX].ensure(2 * cap)) || (e = b[B_BKEY0].ensure(cap * 8)) ||
      (e = b[B_BKEY1].ensure(cap * 8)) || (e = b[B_BVAL0].ensure(cap * 4)) || (e = b[B_BVAL1].ensure(cap * 4)) ||
      (e = b[B_TILECNT].ensure((size_t)nt * 4 * (2 + (kWaveCnt + 1) * (kTile / kSpanRecs)))) ||
      (e = b[B_AD].ensure(cap * (4 + 8 + 8 + 4 + 4 + 4 + 4 + 8 + 1) + 64)) ||
      (e = b[B_K].ensure(cap * (4 + 8 + 8 + 8 + 4 * 4 + 8 + 8 + 8 + 4) + 64)) ||
      (e = b[B_UT].ensure(cap * (4 + 8 + 8 + 8 + 4 + 4 + 8 + 4 + 4 + 1) + 64)) ||
      (e = b[B_WSCAN].ensure((size_t)nt * (kTile / kSpanRecs) * kEp * 8 +
                             (size_t)ceil_div32((size_t)nt * (kTile / kSpanRecs), kScanChunk) * (kWaveCnt * 4 + kEp * 8) + 64)) ||
      (e = b[B_PR].ensure(cap * (4 + 4 + 8 + 8 + 8 + 4) +
                          ((size_t)pair_table_mask((uint32_t)std::min<size_t>(cap / 2, 0x7FFFFFFFu)) + 1) * 12 + 64)) ||
      (e = b[B_HIST].ensure((size_t)kNumJobs * 256 * nt * 4)) ||
      (e = b[B_TOTALS].ensure((size_t)kNumJobs * kMaxPasses * 256 * 4)) ||
      (e = b[B_SEG].ensure((size_t)nt * (kT / 64) * 2 * sizeof(WaveAgg) + 64)) ||
      (e = b[B_SKEY].ensure(cap * 8 * 2 * (kNumJobs - 1) + 64)) || (e = b[B_PARTS].ensure((size_t)kSlots * nt * 8)))
    return e;
  if (!ws->a_side) {
    ODP_HIP(hipStreamCreateWithFlags(&ws->a_side, hipStreamNonBlocking));
    ODP_HIP(hipEventCreateWithFlags(&ws->a_fork, hipEventDisableTiming));
    ODP_HIP(hipEventCreateWithFlags(&ws->a_join, hipEventDisableTiming));
  }
  ws->a_cap_events = cap;
  SortJob hj[kNumJobs];
  build_jobs(views(ws), hj);
  ODP_HIP(hipMemcpy(b[B_JOBS].ptr, hj, sizeof(hj), hipMemcpyHostToDevice));
  return ODP_OK;
}

void analyze_release(Workspace* ws) {
  analyze_drop_graph(ws);
  for (DevBuf& b : ws->a_bufs) b.release();
  ws->a_cap_events = 0;
  if (ws->a_side) {
    (void)hipStreamSynchronize(ws->a_side);
    (void)hipEventDestroy(ws->a_fork);
    (void)hipEventDestroy(ws->a_join);
    (void)hipStreamDestroy(ws->a_side);
    ws->a_side = nullptr;
    ws->a_fork = ws->a_join = nullptr;
  }
}

// ---------------------------------------------------------------------------
// Logs of at most kTinyMax records: the whole analysis in one workgroup, one
// thread per record, each rule written out as its definition. The records sit
// in LDS, compacted into per-class lists (transfers, ALLOC/DELETE, kernels);
// a thread walks the list its rule needs in a loop that is the same for the
// whole wavefront, so every LDS read is a broadcast. One launch, where longer
// logs take 2 (walks), 13 (hash tables) or 76 (sorts).
// ---------------------------------------------------------------------------
constexpr uint32_t kTinyMax = 512;

struct TinyLds {
  unsigned long long dig[kTinyMax], saddr[kTinyMax], daddr[kTinyMax], bytes[kTinyMax], ts[kTinyMax], te[kTinyMax];
  uint16_t list[3][kTinyMax];   // record indices of each class in log order: transfers, ALLOC/DELETE, kernels
  uint16_t del_of[kTinyMax];    // the DELETE paired with an ALLOC
  int8_t src[kTinyMax], dst[kTinyMax];
  uint8_t op[kTinyMax], cls[kTinyMax], paired[kTinyMax];
  uint32_t wcnt[kTinyMax / 64][3];
  unsigned long long acc[kTinyMax / 64][32];
};

enum TinyAcc {
  TA_INV, TA_TX, TA_K, TA_PAIRS, TA_UNP_A, TA_UNP_D, TA_DD, TA_DD_GRP, TA_DD_B, TA_DD_T, TA_RT_TX, TA_RT_RX, TA_RT_B,
  TA_RT_T, TA_RA, TA_RA_GRP, TA_RA_B, TA_RA_T, TA_UA, TA_UA_B, TA_UA_T, TA_UT, TA_UT_B, TA_UT_T, TA_ELIM, TA_TMIN,
  TA_TMAX, TA_BAD, TA_COUNT
};
static_assert(TA_COUNT <= 32, "tiny accumulators");

// The workgroup reduction of each accumulator: the first rejected record and
// the earliest start take the minimum, the latest end the maximum, the rest sum.
__device__ __forceinline__ unsigned long long tiny_red(int k, unsigned long long a, unsigned long long b) {
  return (k == TA_BAD || k == TA_TMIN) ? min(a, b) : k == TA_TMAX ? max(a, b) : a + b;
}

// The report of a whole log from its reduced accumulators.
__device__ void acc_report(const unsigned long long* t, uint32_t n, odp_report* rep) {
  rep->n_events = n;
  rep->n_invalid = t[TA_INV];
  rep->n_transfers = t[TA_TX];
  rep->n_kernels = t[TA_K];
  rep->n_alloc_pairs = t[TA_PAIRS];
  rep->n_unpaired_alloc = t[TA_UNP_A];
  rep->n_unpaired_delete = t[TA_UNP_D];
  rep->dd_events = t[TA_DD];
  rep->dd_groups = t[TA_DD_GRP];
  rep->dd_members = t[TA_DD] + t[TA_DD_GRP];
  rep->dd_bytes = t[TA_DD_B];
  rep->dd_time_ns = t[TA_DD_T];
  rep->rt_pairs = t[TA_RT_TX];
  rep->rt_rx_events = t[TA_RT_RX];
  rep->rt_bytes = t[TA_RT_B];
  rep->rt_time_ns = t[TA_RT_T];
  rep->ra_events = t[TA_RA];
  rep->ra_groups = t[TA_RA_GRP];
  rep->ra_members = t[TA_RA] + t[TA_RA_GRP];
  rep->ra_bytes = t[TA_RA_B];
  rep->ra_time_ns = t[TA_RA_T];
  rep->ua_events = t[TA_UA];
  rep->ua_bytes = t[TA_UA_B];
  rep->ua_time_ns = t[TA_UA_T];
  rep->ut_events = t[TA_UT];
  rep->ut_bytes = t[TA_UT_B];
  rep->ut_time_ns = t[TA_UT_T];
  write_estimate(rep, t[TA_INV] < n, t[TA_TMIN], t[TA_TMAX], t[TA_ELIM]);
  rep->first_bad_event = (uint32_t)t[TA_BAD];
  rep->status = t[TA_BAD] != kNone ? 1 : 0;
}

__global__ __launch_bounds__(kTinyMax) void analyze_tiny_kernel(const odp_event* __restrict__ ev, uint32_t n,
                                                               uint8_t* __restrict__ flags, odp_report* __restrict__ rep) {
  __shared__ TinyLds L;
  const uint32_t i = threadIdx.x;
  const int lane = i & 63, w = i >> 6;
  const bool in = i < n;
  if (in) {
    const odp_event& e = ev[i];
    L.dig[i] = e.digest;
    L.saddr[i] = e.src_addr;
    L.daddr[i] = e.dst_addr;
    L.bytes[i] = e.bytes;
    L.ts[i] = e.t_start;
    L.te[i] = e.t_end;
    L.op[i] = e.op;
    L.src[i] = (int8_t)max(-128, min(127, (int)e.src_dev));
    L.dst[i] = (int8_t)max(-128, min(127, (int)e.dst_dev));
    L.paired[i] = 0;
  }
  __syncthreads();
  // validity (as the classification of longer logs) and the class lists
  uint8_t c = C_INVALID;
  if (in) {
    const uint8_t op = L.op[i];
    const bool tx = op == ODP_H2D || op == ODP_D2H || op == ODP_D2D;
    const bool valid = op >= ODP_ALLOC && op <= ODP_KERNEL && L.te[i] >= L.ts[i] && (i == 0 || L.ts[i] >= L.ts[i - 1]) &&
                       dev_ok(ev[i].dst_dev) && (!tx || dev_ok(ev[i].src_dev));
    if (valid) c = tx ? C_TRANSFER : op == ODP_KERNEL ? C_KERNEL : C_ALLOCDEL;
    L.cls[i] = c;
  }
  uint32_t pos[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const uint64_t m = __ballot(c == C_TRANSFER + k);
    pos[k] = (uint32_t)__popcll(m & lanemask_lt());
    if (lane == 0) L.wcnt[w][k] = (uint32_t)__popcll(m);
  }
  __syncthreads();
  uint32_t cnt[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    uint32_t before = 0, all = 0;
    for (int x = 0; x < (int)(kTinyMax / 64); ++x) {
      if (x < w) before += L.wcnt[x][k];
      all += L.wcnt[x][k];
    }
    cnt[k] = all;
    if (c == C_TRANSFER + k) L.list[k][before + pos[k]] = (uint16_t)i;
  }
  __syncthreads();
  unsigned long long a[TA_COUNT];
#pragma unroll
  for (int k = 0; k < TA_COUNT; ++k) a[k] = 0;
  a[TA_BAD] = in && c == C_INVALID ? i : kNone;
  a[TA_TMIN] = in && c != C_INVALID ? L.ts[i] : ~0ull;
  a[TA_TMAX] = in && c != C_INVALID ? L.te[i] : 0ull;
  a[TA_INV] = in && c == C_INVALID;
  a[TA_TX] = c == C_TRANSFER;
  a[TA_K] = c == C_KERNEL;
  uint8_t f = in && c == C_INVALID ? ODP_F_INVALID : 0;
  // duplicates and round trips: one walk over the transfers
  if (c == C_TRANSFER) {
    const unsigned long long dg = L.dig[i];
    const int sr = L.src[i], ds = L.dst[i];
    bool dd = false, later = false, tx = false, rx = false;
#pragma unroll 4
    for (uint32_t q = 0; q < cnt[0]; ++q) {
      const uint32_t j = L.list[0][q];
      if (L.dig[j] != dg) continue;
      const int sj = L.src[j], dj = L.dst[j];
      if (j < i) {
        dd |= dj == ds;
        // the latest earlier transfer between the same two endpoints (the walk is in log order)
        if (sr != ds && sj != dj && ((sj == sr && dj == ds) || (sj == ds && dj == sr))) rx = sj == ds;
      } else if (j > i) {
        later |= dj == ds;
        tx |= sr != ds && sj == ds && dj == sr;
      }
    }
    const unsigned long long b = L.bytes[i], d = L.te[i] - L.ts[i];
    if (dd) {
      f |= ODP_F_DD;
      a[TA_DD] = 1;
      a[TA_DD_B] = b;
      a[TA_DD_T] = d;
    } else {
      a[TA_DD_GRP] = later;
    }
    if (tx) {
      f |= ODP_F_RT_TX;
      a[TA_RT_TX] = 1;
    }
    if (rx) {
      f |= ODP_F_RT_RX;
      a[TA_RT_RX] = 1;
      a[TA_RT_B] = b;
      a[TA_RT_T] = d;
    }
    // unused transfer: a copy into device memory that no kernel on the device
    // meets between its start and the start of the next copy to the same
    // (receiver, sender, source address)
    if (L.op[i] != ODP_D2H && ds >= 0) {
      const unsigned long long sa = L.saddr[i];
      unsigned long long hi = ~0ull;
      bool found = false;
#pragma unroll 4
      for (uint32_t q = 0; q < cnt[0]; ++q) {
        const uint32_t j = L.list[0][q];
        if (!found && j > i && L.op[j] != ODP_D2H && L.dst[j] == ds && L.src[j] == sr && L.saddr[j] == sa) {
          hi = L.ts[j];
          found = true;
        }
      }
      const unsigned long long lo = L.ts[i];
      bool read = false;
#pragma unroll 4
      for (uint32_t q = 0; q < cnt[2]; ++q) {
        const uint32_t k = L.list[2][q];
        read |= L.dst[k] == ds && L.ts[k] <= hi && L.te[k] >= lo;
      }
      if (!read) {
        f |= ODP_F_UT;
        a[TA_UT] = 1;
        a[TA_UT_B] = b;
        a[TA_UT_T] = d;
      }
    }
    if (f & (ODP_F_DD | ODP_F_RT_RX | ODP_F_UT)) a[TA_ELIM] = d;
  }
  // pairing: a DELETE pairs with the record just before it in its (device,
  // device address) group when that record is an ALLOC
  if (c == C_ALLOCDEL && L.op[i] == ODP_DELETE) {
    const int ds = L.dst[i];
    const unsigned long long da = L.daddr[i];
    uint32_t prev = kNone;
#pragma unroll 4
    for (uint32_t q = 0; q < cnt[1]; ++q) {
      const uint32_t j = L.list[1][q];
      if (j < i && L.dst[j] == ds && L.daddr[j] == da) prev = j;
    }
    if (prev != kNone && L.op[prev] == ODP_ALLOC) {
      L.paired[prev] = 1;
      L.del_of[prev] = (uint16_t)i;
      L.paired[i] = 1;
    }
  }
  __syncthreads();
  if (c == C_ALLOCDEL) {
    if (L.paired[i]) {
      f |= ODP_F_PAIRED;
    } else if (L.op[i] == ODP_ALLOC) {
      a[TA_UNP_A] = 1;
    } else {
      a[TA_UNP_D] = 1;
    }
  }
  // repeated and unused allocations, over the paired ALLOCs
  if (c == C_ALLOCDEL && L.paired[i] && L.op[i] == ODP_ALLOC) {
    const uint32_t del = L.del_of[i];
    const int ds = L.dst[i];
    const unsigned long long ha = L.saddr[i], b = L.bytes[i];
    bool ra = false, later = false;
#pragma unroll 4
    for (uint32_t q = 0; q < cnt[1]; ++q) {
      const uint32_t j = L.list[1][q];
      if (j == i || L.op[j] != ODP_ALLOC || !L.paired[j]) continue;
      if (L.saddr[j] == ha && L.dst[j] == ds && L.bytes[j] == b) {
        ra |= j < i;
        later |= j > i;
      }
    }
    const unsigned long long t0 = L.ts[i], t1 = L.te[del];
    bool used = false;
#pragma unroll 4
    for (uint32_t q = 0; q < cnt[2]; ++q) {
      const uint32_t k = L.list[2][q];
      used |= L.dst[k] == ds && L.ts[k] <= t1 && L.te[k] >= t0;
    }
    const unsigned long long d = (L.te[i] - L.ts[i]) + (L.te[del] - L.ts[del]);
    a[TA_PAIRS] = 1;
    if (ra) {
      f |= ODP_F_RA;
      a[TA_RA] = 1;
      a[TA_RA_B] = b;
      a[TA_RA_T] = d;
    } else {
      a[TA_RA_GRP] = later;
    }
    if (!used) {
      f |= ODP_F_UA;
      a[TA_UA] = 1;
      a[TA_UA_B] = b;
      a[TA_UA_T] = d;
    }
    if (ra || !used) a[TA_ELIM] = d;
  }
  if (in) flags[i] = f;
  // the report: sums (the first rejected record: minimum) over the workgroup
#pragma unroll
  for (int k = 0; k < TA_COUNT; ++k) {
    unsigned long long v = a[k];
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v = tiny_red(k, v, __shfl_xor(v, o, 64));
    if (lane == 0) L.acc[w][k] = v;
  }
  __syncthreads();
  if (i < TA_COUNT) {  // one thread per field folds the wavefronts' partials
    unsigned long long v = L.acc[0][i];
#pragma unroll
    for (int x = 1; x < (int)(kTinyMax / 64); ++x) v = tiny_red((int)i, v, L.acc[x][i]);
    L.acc[0][i] = v;
  }
  __syncthreads();
  if (i == 0) {
    acc_report(L.acc[0], n, rep);
  }
}

// ---------------------------------------------------------------------------
// Logs of kTinyMax + 1 .. kWalkMax records: every rule evaluated as its
// definition here too, by all workgroups. What a record needs to know about
// the others is a maximum, a minimum, an OR or a count over them, so the
// others may be looked at in any order and by several lanes: a workgroup
// stages the whole log's keys in LDS and takes 16 records, each with 64 lanes
// that walk every 64th record; the partial results meet in LDS. Two launches on
// one stream:
//   walk   DD, RT, the next copy and UT, pairing and UA
//   pairs  RA over the paired ALLOCs; the report by the last workgroup
// instead of the sorting pipeline's 26 (up to 2,048 records) or 79, each bound
// by its latency. The work grows with n^2, and 4,096 records fill the LDS:
// 1,000 records 145 -> 21 us, 4,000 records 224 -> 40 us.
// ---------------------------------------------------------------------------
constexpr int kWalkT = 1024;
constexpr uint32_t kWalkRec = 16;                     // records per workgroup
constexpr uint32_t kWalkSub = kWalkT / kWalkRec;      // lanes per record
constexpr uint32_t kUnusedBit = 0x80000000u;          // in pair[]: no kernel meets the pair's window
constexpr uint32_t kNoGroup = 0xFFFFFFFFu;

struct WalkKeys {
  unsigned long long k1, k2;  // transfers: digest, source address; ALLOC/DELETE: -, device address; KERNELs: start, end
};
struct WalkCode {
  uint32_t m;  // 0 rejected; else bit 3, bit 0 transfer, bit 1 KERNEL, bit 2 DELETE, src_dev + 1 << 8; dst_dev + 1 << 12
  uint32_t g;  // with k2, the group of copies into one place or of one device address; 0 for other records
};

struct WalkArgs {
  const odp_event* ev;
  uint32_t n;
  uint8_t* flags;
  odp_report* rep;
  uint32_t* pair;            // per record: an ALLOC's DELETE (| kUnusedBit), else kNone
  unsigned long long* sums;  // [2 * workgroups][kWalkAcc] accumulators of the walk's and the pairs' workgroups
  AnaCtl* ctl;               // wticket
};
constexpr uint32_t kWalkAcc = 32;

__device__ __forceinline__ unsigned long long acc_identity(int k) {
  return k == TA_BAD ? (unsigned long long)kNone : k == TA_TMIN ? ~0ull : 0ull;
}

__global__ __launch_bounds__(kWalkT) void walk_kernel(WalkArgs A) {
  __shared__ WalkKeys s_key[kWalkMax];
  __shared__ WalkCode s_code[kWalkMax];
  __shared__ uint16_t s_k[kWalkMax];  // the KERNEL records, in any order
  __shared__ uint32_t s_nk;
  __shared__ uint32_t s_fl[kWalkRec], s_rx[kWalkRec], s_next[kWalkRec], s_prev[kWalkRec], s_cnt[kWalkRec];
  __shared__ unsigned long long s_lo[kWalkRec], s_hi[kWalkRec];
  __shared__ unsigned long long s_acc[kWalkAcc][kWalkRec];
  const odp_event* __restrict__ ev = A.ev;
  const uint32_t n = A.n, t = threadIdx.x, lane = t & 63, w = t >> 6;
  if (blockIdx.x == 0 && t == 0) A.ctl->wticket = 0;
  if (t == 0) s_nk = 0;
  if (t < kWalkRec) {
    s_fl[t] = s_rx[t] = s_prev[t] = s_cnt[t] = 0;
    s_next[t] = kNone;
  }
  if (t < kWalkAcc * kWalkRec) s_acc[t / kWalkRec][t % kWalkRec] = acc_identity((int)(t / kWalkRec));
  __syncthreads();
  // every record's keys and codes
  for (uint32_t j = t; j < n; j += kWalkT) {
    const odp_event e = ev[j];
    const uint64_t before = j ? ev[j - 1].t_start : 0;
    const bool tx = e.op == ODP_H2D || e.op == ODP_D2H || e.op == ODP_D2D;
    const bool valid = e.op >= ODP_ALLOC && e.op <= ODP_KERNEL && e.t_end >= e.t_start && e.t_start >= before &&
                       dev_ok(e.dst_dev) && (!tx || dev_ok(e.src_dev));
    const bool kern = valid && e.op == ODP_KERNEL, ad = valid && !tx && !kern;
    const bool copyin = valid && tx && e.op != ODP_D2H && e.dst_dev >= 0;
    const uint32_t sd = tx ? (uint32_t)(e.src_dev + 1) : 0u, dd = (uint32_t)(e.dst_dev + 1);
    s_key[j] = kern ? WalkKeys{e.t_start, e.t_end} : WalkKeys{e.digest, ad ? e.dst_addr : e.src_addr};
    s_code[j] = WalkCode{!valid ? 0u : 8u | (tx ? 1u : 0u) | (kern ? 2u : 0u) | (e.op == ODP_DELETE ? 4u : 0u) | sd << 8 | dd << 12,
                         copyin ? 1u | sd << 8 | dd << 12 : ad ? 2u | dd << 12 : 0u};
    const uint64_t bk = __ballot(kern);
    if (bk) {
      uint32_t q = 0;
      if (lane == (uint32_t)__builtin_ctzll(bk)) q = atomicAdd(&s_nk, (uint32_t)__popcll(bk));
      q = (uint32_t)__shfl((int)q, __builtin_ctzll(bk), 64) + (uint32_t)__popcll(bk & lanemask_lt());
      if (kern) s_k[q] = (uint16_t)j;
    }
  }
  __syncthreads();
  const uint32_t r = lane % kWalkRec, sub = w * (64 / kWalkRec) + lane / kWalkRec, i = blockIdx.x * kWalkRec + r;
  const bool in = i < n;
  const WalkKeys ki = in ? s_key[i] : WalkKeys{0, 0};
  const WalkCode ci = in ? s_code[i] : WalkCode{0, 0};
  const bool tx = ci.m & 1;
  const uint32_t sr = (ci.m >> 8) & 15, ds = (ci.m >> 12) & 15, gi = ci.g ? ci.g : kNoGroup;
  // rx: 1 + 2 * (latest earlier transfer of the pair) + whether it went the
  // other way; prev, next: the nearest records of i's group (prev plus 1)
  uint32_t fl = 0, rx = 0, next = kNone, prev = 0;
#pragma unroll 4
  for (uint32_t j = sub; j < n; j += kWalkSub) {
    const WalkKeys kj = s_key[j];
    const WalkCode cj = s_code[j];
    if (kj.k1 == ki.k1 && tx && (cj.m & 1)) {
      const uint32_t sj = (cj.m >> 8) & 15, dj = (cj.m >> 12) & 15;
      if (j < i) {
        fl |= dj == ds ? 1u : 0u;
        if (sr != ds && ((sj == sr && dj == ds) || (sj == ds && dj == sr))) rx = 1 + 2 * j + (sj == ds ? 1u : 0u);
      } else if (j > i) {
        fl |= (dj == ds ? 2u : 0u) | (sr != ds && sj == ds && dj == sr ? 4u : 0u);
      }
    }
    if (kj.k2 == ki.k2 && cj.g == gi) {
      if (j < i) prev = 1 + j;
      if (j > i) next = min(next, j);
    }
  }
  if (fl) atomicOr(&s_fl[r], fl);
  if (rx) atomicMax(&s_rx[r], rx);
  if (next != kNone) atomicMin(&s_next[r], next);
  if (prev) atomicMax(&s_prev[r], prev);
  __syncthreads();
  // The window the device's kernels are counted over: of a copy into the
  // device, or of the pair that an ALLOC opens.
  const bool del = ci.m & 4, ad = (ci.g & 3) == 2, copyin = (ci.g & 3) == 1;
  const uint32_t nx = s_next[r];
  const bool alloc_paired = ad && !del && nx != kNone && (s_code[nx == kNone ? 0 : nx].m & 4);
  odp_event e{};
  if (t < kWalkRec && in) {
    e = ev[i];
    s_lo[r] = e.t_start;
    s_hi[r] = alloc_paired ? ev[nx].t_end : nx == kNone ? ~0ull : ev[nx].t_start;
  }
  __syncthreads();
  // kernels on the device that start by the window's end, less those that end
  // before it opens
  if (copyin || alloc_paired) {
    const uint64_t lo = s_lo[r], hi = s_hi[r];
    const uint32_t nk = s_nk;
    uint32_t cnt = 0;
#pragma unroll 2
    for (uint32_t q = sub; q < nk; q += kWalkSub) {
      const uint32_t j = s_k[q];
      const WalkKeys kj = s_key[j];
      if (((s_code[j].m >> 12) & 15) == ds) cnt += (kj.k1 <= hi ? 1u : 0u) - (kj.k2 < lo ? 1u : 0u);
    }
    if (cnt) atomicAdd(&s_cnt[r], cnt);
  }
  __syncthreads();
  if (t < kWalkRec && in) {
    const bool unread = s_cnt[r] == 0;
    const unsigned long long d = e.t_end - e.t_start;
    uint8_t f = 0;
    uint32_t pr = kNone;
    if (!ci.m) {
      f = ODP_F_INVALID;
      s_acc[TA_INV][r] = 1;
      s_acc[TA_BAD][r] = i;
    } else {
      s_acc[TA_TMIN][r] = e.t_start;
      s_acc[TA_TMAX][r] = e.t_end;
    }
    if (tx) {
      s_acc[TA_TX][r] = 1;
      const uint32_t x = s_fl[r];
      if (x & 1) {
        f |= ODP_F_DD;
        s_acc[TA_DD][r] = 1;
        s_acc[TA_DD_B][r] = e.bytes;
        s_acc[TA_DD_T][r] = d;
      } else {
        s_acc[TA_DD_GRP][r] = (x >> 1) & 1;
      }
      if (x & 4) {
        f |= ODP_F_RT_TX;
        s_acc[TA_RT_TX][r] = 1;
      }
      if (s_rx[r] && ((s_rx[r] - 1) & 1)) {
        f |= ODP_F_RT_RX;
        s_acc[TA_RT_RX][r] = 1;
        s_acc[TA_RT_B][r] = e.bytes;
        s_acc[TA_RT_T][r] = d;
      }
      if (copyin && unread) {
        f |= ODP_F_UT;
        s_acc[TA_UT][r] = 1;
        s_acc[TA_UT_B][r] = e.bytes;
        s_acc[TA_UT_T][r] = d;
      }
      if (f & (ODP_F_DD | ODP_F_RT_RX | ODP_F_UT)) s_acc[TA_ELIM][r] = d;
    } else if (ci.m & 2) {
      s_acc[TA_K][r] = 1;
    } else if (ad && del) {
      const uint32_t pv = s_prev[r];
      const bool paired = pv && !(s_code[pv ? pv - 1 : 0].m & 4);
      f = paired ? ODP_F_PAIRED : 0;
      s_acc[TA_UNP_D][r] = !paired;
    } else if (ad) {
      s_acc[TA_UNP_A][r] = !alloc_paired;
      if (alloc_paired) pr = nx | (unread ? kUnusedBit : 0u);
    }
    A.flags[i] = f;  // (a paired ALLOC's flags follow in the pairs kernel)
    A.pair[i] = pr;
  }
  __syncthreads();
  if (t < kWalkAcc) {
    unsigned long long v = s_acc[t][0];
    for (uint32_t x = 1; x < kWalkRec; ++x) v = tiny_red((int)t, v, s_acc[t][x]);
    A.sums[(size_t)blockIdx.x * kWalkAcc + t] = v;
  }
}

// One workgroup per 64 records, for the paired ALLOCs among them; the walked
// records are spread over its wavefronts. The last workgroup to finish folds
// all sums into the report.
constexpr uint32_t kWalkPairRec = 64;
__global__ __launch_bounds__(kWalkT) void walk_pairs_kernel(WalkArgs A, uint32_t walk_blocks) {
  __shared__ uint32_t s_list[kWalkMax];  // the paired ALLOCs of the log, in any order
  __shared__ uint32_t s_n, s_fl[kWalkPairRec], s_last;
  __shared__ unsigned long long s_part[kWalkT / kWalkAcc][kWalkAcc];
  const odp_event* __restrict__ ev = A.ev;
  const uint32_t n = A.n, t = threadIdx.x, lane = t & 63, w = t >> 6;
  const uint32_t i = blockIdx.x * kWalkPairRec + lane;
  const uint32_t pr = i < n ? A.pair[i] : kNone;
  unsigned long long* own = A.sums + (size_t)(walk_blocks + blockIdx.x) * kWalkAcc;
  unsigned long long a[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
  const bool any = __ballot(pr != kNone) != 0;  // the same 64 records in every wavefront
  if (any) {
    if (t == 0) s_n = 0;
    if (t < kWalkPairRec) s_fl[t] = 0;
    __syncthreads();
    for (uint32_t j = t; j < n; j += kWalkT) {
      const uint64_t b = __ballot(A.pair[j] != kNone);
      if (!b) continue;
      uint32_t q = 0;
      if (lane == (uint32_t)__builtin_ctzll(b)) q = atomicAdd(&s_n, (uint32_t)__popcll(b));
      q = (uint32_t)__shfl((int)q, __builtin_ctzll(b), 64) + (uint32_t)__popcll(b & lanemask_lt());
      if ((b >> lane) & 1) s_list[q] = j;
    }
    odp_event e{};
    if (pr != kNone) e = ev[i];
    __syncthreads();
    const uint32_t np = s_n;
    uint32_t fl = 0;  // 1: an earlier paired ALLOC of the key, 2: a later one
    // 64 listed ALLOCs at a time, one per lane, handed round by lane reads
    for (uint32_t q0 = w * 64; q0 < np; q0 += kWalkT) {
      const bool ok = q0 + lane < np;
      const uint32_t jl = ok ? s_list[q0 + lane] : 0u;
      const uint64_t hl = ok ? ev[jl].src_addr : 0ull, bl = ok ? ev[jl].bytes : 0ull;
      const int dl = ok ? ev[jl].dst_dev : -2;
      const int m = (int)min(64u, np - q0);
      for (int x = 0; x < m; ++x) {
        const uint32_t j = lane32(jl, x);
        if (lane64(hl, x) == e.src_addr && lane64(bl, x) == e.bytes && (int)lane32((uint32_t)dl, x) == e.dst_dev)
          fl |= j < i ? 1u : j > i ? 2u : 0u;
      }
    }
    if (fl && pr != kNone) atomicOr(&s_fl[lane], fl);
    __syncthreads();
    if (t < 64 && pr != kNone) {
      const odp_event& ed = ev[pr & ~kUnusedBit];
      const unsigned long long d = (e.t_end - e.t_start) + (ed.t_end - ed.t_start);
      uint8_t f = ODP_F_PAIRED;
      a[0] = 1;
      if (s_fl[lane] & 1) {
        f |= ODP_F_RA;
        a[1] = 1;
        a[3] = e.bytes;
        a[4] = d;
      } else {
        a[2] = s_fl[lane] >> 1;
      }
      if (pr & kUnusedBit) {
        f |= ODP_F_UA;
        a[5] = 1;
        a[6] = e.bytes;
        a[7] = d;
      }
      if (f & (ODP_F_RA | ODP_F_UA)) a[8] = d;
      A.flags[i] = f;
    }
  }
  if (t < 64) {
    // this workgroup's sums, and after them its ticket
    constexpr int kAcc[9] = {TA_PAIRS, TA_RA, TA_RA_GRP, TA_RA_B, TA_RA_T, TA_UA, TA_UA_B, TA_UA_T, TA_ELIM};
    unsigned long long mine = acc_identity((int)lane);
    if (any) {
#pragma unroll
      for (int k = 0; k < 9; ++k) {
        const unsigned long long v = wave_sum(a[k]);
        if ((int)lane == kAcc[k]) mine = v;
      }
    }
    if (lane < kWalkAcc) __hip_atomic_store(own + lane, mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (t == 0)
      s_last = __hip_atomic_fetch_add(&A.ctl->wticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1;
  }
  __syncthreads();
  if (!s_last) return;
  const uint32_t k = t % kWalkAcc, part = t / kWalkAcc;
  unsigned long long v = acc_identity((int)k);
  for (uint32_t b = part; b < walk_blocks + gridDim.x; b += kWalkT / kWalkAcc)
    v = tiny_red((int)k, v, __hip_atomic_load(A.sums + (size_t)b * kWalkAcc + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
  s_part[part][k] = v;
  __syncthreads();
  if (t < kWalkAcc) {
    for (uint32_t x = 1; x < kWalkT / kWalkAcc; ++x) v = tiny_red((int)t, v, s_part[x][t]);
    s_part[0][t] = v;
  }
  __syncthreads();
  if (t == 0) acc_report(s_part[0], n, A.rep);
}

// Digest passes to run before the first local fix, for n records (at most n
// distinct digests): the least k with 2^(8k) >= 16 n, so that a run of equal
// low bytes holds on average at most 1/16 of a digest besides its own and the
// local sorts (a few, short) replace the remaining passes.
uint32_t first_digest_passes(size_t n) {
  uint32_t k = 1;
  while (k < 8 && std::ldexp(1.0, 8 * (int)k) < 16.0 * (double)n) ++k;
  return k;
}

}  // namespace odp

using namespace odp;

// The launch sequence of one analysis of 1 .. kMidMax records.
static int enqueue_mid(Workspace* ws, const odp_event* events, size_t n, uint8_t* out_flags, odp_report* out_report,
                       hipStream_t stream, uint32_t* alg2_rx, unsigned long long* alg2_np) {
  const Views v = views(ws);
  const MidView& m = v.mid;
  const uint32_t nn = (uint32_t)n, tiles = ceil_div32(n, kMidTile), blocks = ceil_div32(n, kT * kMidRounds),
                 cblocks = ceil_div32(n, kClsT * kClsRounds);
  AnaCtl* ctl = v.ctl;
  // digest table: at most half full; its slot numbers split into two digits
  uint32_t tb = 10;
  while ((1ull << tb) < 2 * n) ++tb;
  const uint32_t bits = (tb + 1) / 2;
  static_assert(kMidMax <= 1u << 18 && kMidDigits >= 1u << 10, "two digits cover the table");

  if (alg2_rx)
    hipLaunchKernelGGL(alg2_fill_kernel, dim3(ceil_div32(n, kT)), dim3(kT), 0, stream, alg2_rx, nn, alg2_np);
  hipLaunchKernelGGL(mid_clear_kernel, dim3(std::max<uint32_t>(1, (1u << tb) / (4 * kMidT))), dim3(kMidT), 0, stream, m.dtab,
                     1u << tb, m.h0, tiles << bits, ctl, nn);
  MidClassify C;
  C.ev = events;
  C.n = nn;
  C.flags = out_flags;
  C.cls = v.cls;
  C.uth = m.uth;
  C.gid = m.gid0;
  C.val = v.bv[0];
  C.wave_cnt = m.wscan.cnt;
  C.wave_kmax = m.wscan.kmax;
  C.dtab = m.dtab;
  C.dmask = (1u << tb) - 1;
  C.hist = m.h0;
  C.bits = bits;
  C.parts = m.parts;
  hipLaunchKernelGGL(mid_classify_kernel, dim3(cblocks), dim3(kClsT), 0, stream, C);
  WaveScan W = m.wscan;
  W.nw = cblocks * (kClsT / 64);
  const uint32_t nchunk = ceil_div32(W.nw, kScanChunk);
  hipLaunchKernelGGL(mid_scan_kernel, dim3(nchunk * kScanQ + kMidSums), dim3(kMidT), 0, stream, W, nchunk, ctl, m.parts,
                     cblocks, out_report, v.jobs + kJobBig);

  // Fork: as in the pipeline for longer logs.
  hipStream_t side = ws->a_side;
  ODP_HIP(hipEventRecord(ws->a_fork, stream));
  ODP_HIP(hipStreamWaitEvent(side, ws->a_fork, 0));
  MidSide A;
  A.ev = events;
  A.cls = v.cls;
  A.n = nn;
  A.W = W;
  A.S = v.S;
  A.M = m;
  A.T = v.pt;
  A.flags = out_flags;
  A.ctl = ctl;
  UtArgs& U = A.U;
  U = UtArgs{};
  U.ev = events;
  U.n_ut = &ctl->n_ut;
  U.ut_idx = v.S.ut_idx;
  U.ut_w_addr = v.S.ut_w_addr;
  U.ut_w_code = v.S.ut_w_code;
  U.ut_ts = v.S.ut_ts;
  U.ut_kc = v.S.ut_kc;
  U.ut_km = v.S.ut_km;
  U.ut_hit = v.ut_hit;
  U.kd_ts = v.S.kd_ts;
  U.kd_idx = v.S.kd_idx;
  U.ctl = ctl;
  // (in turn: the host enqueues about as fast as the device runs)
  hipLaunchKernelGGL(mid_subset_kernel, dim3(cblocks), dim3(kT), 0, side, A);
  hipLaunchKernelGGL(mid_scatter_kernel, dim3(tiles), dim3(kMidT), 0, stream, 0u, nn, ctl, bits, m.h0, m.gid0, v.bv[0], m.gid1,
                     nullptr, v.bv[1]);
  hipLaunchKernelGGL(mid_link_kernel, dim3(2 * blocks), dim3(kT), 0, side, A);
  hipLaunchKernelGGL(mid_hist_kernel, dim3(tiles), dim3(kMidT), 0, stream, ctl, bits, m.gid1, m.h1);
  hipLaunchKernelGGL(mid_pair_kernel, dim3(blocks), dim3(kT), 0, side, A);
  hipLaunchKernelGGL(mid_scatter_kernel, dim3(tiles), dim3(kMidT), 0, stream, 1u, nn, ctl, bits, m.h1, m.gid1, v.bv[1], nullptr,
                     v.bk[0], v.bv[0]);
  hipLaunchKernelGGL(mid_ra_ua_kernel, dim3(blocks), dim3(kT), 0, side, A);
  ODP_HIP(hipEventRecord(ws->a_join, side));
  DDArgs D{};
  D.ev = events;
  D.n = nn;
  D.aux = v.aux;
  D.job = v.jobs + kJobBig;
  D.ctl = ctl;
  D.agg = m.agg;
  D.flags = out_flags;
  D.rep = out_report;
  D.parts = m.parts;
  D.uth = m.uth;
  hipLaunchKernelGGL(ddrt_agg_kernel<kMidRounds>, dim3(blocks), dim3(kT), 0, stream, D);
  if (alg2_rx) {
    Alg2Args G{};
    G.job = v.jobs + kJobBig;
    G.aux = v.aux;
    G.n = nn;
    G.rx = alg2_rx;
    G.npairs = alg2_np;
    hipLaunchKernelGGL(alg2_kernel, dim3(ceil_div32(n, kT)), dim3(kT), 0, stream, G);
  }
  ODP_HIP(hipStreamWaitEvent(stream, ws->a_join, 0));
  hipLaunchKernelGGL((ddrt_final_kernel<kMidRounds, true>), dim3(blocks), dim3(kT), 0, stream, D);
  hipLaunchKernelGGL(mid_finish_kernel, dim3(1), dim3(kMidT), 0, stream, m.parts, blocks, blocks, nn, ctl, out_report);
  return check_hip(hipGetLastError(), "odp_analyze_trace launch");
}

// The launch sequence of one analysis (with the literal Algorithm 2 pairs when
// alg2_rx / alg2_np are given), in the workspace `ws` (reserved for n), enqueued
// on `stream`.
static int enqueue_analysis(Workspace* ws, const odp_event* events, size_t n, uint8_t* out_flags,
                            odp_report* out_report, hipStream_t stream, uint32_t* alg2_rx = nullptr,
                            unsigned long long* alg2_np = nullptr) {
  if (n > 0 && n <= kMidMax) return enqueue_mid(ws, events, n, out_flags, out_report, stream, alg2_rx, alg2_np);
  const Views v = views(ws);
  const uint32_t nn = (uint32_t)n;
  const uint32_t nt = n ? ceil_div32(n, kTile) : 1;  // tiles of this call
  const int cus = cu_count(ws->device);
  const uint32_t grid_map = std::min<uint32_t>(nt * 4, (uint32_t)cus * 8);
  // grid-stride launches whose blocks store one partial per sum (at most one
  // per tile: the partials' row length)
  const uint32_t grid_sum = std::min<uint32_t>(nt, (uint32_t)cus * 8);
  // one thread per element of a subset of at most n (copy-ins) or n / 2
  // (pairs) elements, for the per-element kernels that wait on chains of
  // dependent loads and add nothing up per block: they overlap those waits
  // across many more waves than a grid-stride loop over grid_map blocks does
  const uint32_t grid_rec = n ? ceil_div32(n, kT) : 1, grid_pair = ceil_div32(n / 2 + 1, kT);
  AnaCtl* ctl = v.ctl;

  if (alg2_rx)
    hipLaunchKernelGGL(alg2_fill_kernel, dim3(n ? ceil_div32(n, kT) : 1), dim3(kT), 0, stream, alg2_rx, nn, alg2_np);
  if (n == 0) {
    hipLaunchKernelGGL(init_kernel, dim3(64), dim3(kT), 0, stream, ctl, out_report, v.totals);
    hipLaunchKernelGGL(finalize_kernel, dim3(1), dim3(kT), 0, stream, v.parts, 0u, ctl, out_report);
    return check_hip(hipGetLastError(), "odp_analyze_trace launch");
  }
  hipLaunchKernelGGL(classify_kernel, dim3(nt), dim3(kClassT), 0, stream, events, nn, out_flags, v.cls, v.aux, v.bk[0],
                     v.bv[0], v.wave_cnt, v.wave_copies, v.wscan.kmax, v.hist + (size_t)kJobBig * 256 * v.ntc, v.ntc,
                     alg2_rx ? nullptr : v.cand, v.parts, ctl, out_report, v.totals);
  // the classification's counts, digest masks, first rejected record and endpoint range
  // (the digest sort is planned from them; the literal Algorithm 2 pairs a
  // self-transfer with itself, so there the single digests stay)
  const JobSet Jb{v.jobs + kJobBig, 1, nt};
  const uint32_t kfirst = first_digest_passes(n);
  const bool filter = alg2_rx == nullptr;
  const PlanArgs plan_none{};
  const PlanArgs plan_big{Jb, kfirst, filter ? v.cand : nullptr, filter ? &ctl->n_cand : nullptr, &ctl->plan_ticket[0]};
  hipLaunchKernelGGL(reduce_parts_kernel, dim3(S_AD_DEV_OR), dim3(kT), 0, stream, v.parts, nt, 0u, ctl, out_report, plan_big);

  // Fork: the allocation path (subsets, their sorts, pairing, RA/UA) runs on
  // the workspace's side stream while the digest groups are sorted and
  // scanned on the caller's stream; joined before the report is finished.
  hipStream_t side = ws->a_side;
  ODP_HIP(hipEventRecord(ws->a_fork, stream));
  ODP_HIP(hipStreamWaitEvent(side, ws->a_fork, 0));

  // The allocation path on the side stream, enqueued first (it waits only
  // for the classification), then the digest path on the caller's stream.
  WaveScan WS = v.wscan;
  WS.nw = nt * (kTile / kSpanRecs);
  WS.copies = v.wave_copies;
  const uint32_t nchunk = ceil_div32(WS.nw, kScanChunk);
  hipLaunchKernelGGL(wave_scan_kernel, dim3(nchunk * kScanQ), dim3(1024), 0, side, WS, nchunk, ctl);
  hipLaunchKernelGGL(subset_scatter_kernel, dim3(nt), dim3(kT), 0, side, events, v.cls, nn, WS, v.S, v.parts);
  // Unused transfers (their flags are merged after the join).
  UtArgs U;
  U.ev = events;
  U.n = nn;
  U.cls = v.cls;
  U.W = WS;
  U.ut_job = v.jobs + kJobUt;
  U.n_ut = &ctl->n_ut;
  U.ut_idx = v.S.ut_idx;
  U.ut_w_addr = v.S.ut_w_addr;
  U.ut_w_code = v.S.ut_w_code;
  U.ut_ts = v.S.ut_ts;
  U.ut_kc = v.S.ut_kc;
  U.ut_km = v.S.ut_km;
  U.starts_sorted = v.starts_sorted;
  U.ends_sorted = v.ends_sorted;
  U.next_q = v.next_q;
  U.ut_hit = v.ut_hit;
  U.kd_ts = v.S.kd_ts;
  U.kd_idx = v.S.kd_idx;
  U.ctl = ctl;
  U.flags = out_flags;
  U.parts = v.parts;
  hipLaunchKernelGGL(ut_scan_kernel, dim3(grid_rec), dim3(kT), 0, side, U);
  // ALLOC/DELETE by (device, address), kernels by (device, start) and (device,
  // end), copy-ins by (endpoints, source address). The subsets are usually
  // far smaller than the log: a capped number of blocks per job loops over
  // its tiles instead of a block per log tile.
  const uint32_t side_blocks = std::min<uint32_t>(nt, (uint32_t)cus * 2);
  const JobSet Js{v.jobs + kJobAd, kSubsetJobs, side_blocks};
  const PlanArgs plan_side{Js, 0u, nullptr, nullptr, &ctl->plan_ticket[1]};
  hipLaunchKernelGGL(reduce_parts_kernel, dim3(S_DD_EVENTS - S_AD_DEV_OR), dim3(kT), 0, side, v.parts, nt,
                     (uint32_t)S_AD_DEV_OR, ctl, out_report, plan_side);
  for (uint32_t p = 0; p < 9; ++p) {
    hipLaunchKernelGGL(sort_hist_kernel, dim3(Js.njobs * side_blocks), dim3(kT), 0, side, Js, p);
    hipLaunchKernelGGL(sort_scan_kernel, dim3(256 * Js.njobs), dim3(kT), 0, side, Js, p);
    hipLaunchKernelGGL(sort_scatter_kernel, dim3(Js.njobs * side_blocks), dim3(kST), 0, side, Js, p);
  }
  // Meanwhile the records by digest, up to 8 passes, on the caller's stream.
  // Only the launches after the sorts alternate between the two streams, so that
  // neither chain waits for the other's to be enqueued (1 million records 386 ->
  // 355 us). Alternating from the first pass on takes 355 us there and 558
  // instead of 517 for 2 million records on 8 devices, whose subsets sort longer.
  const uint32_t nft = (uint32_t)((n + kFixTile - 1) / kFixTile);  // tiles of the local fix
  // the digest histograms take two tiles per block on long logs (measured a
  // little faster than one: the per-block start-up is amortised)
  const JobSet Jh{v.jobs + kJobBig, 1, nt > 4u * (uint32_t)cus ? (nt + 1) / 2 : nt};
  for (uint32_t p = 0; p < 8; ++p) {
    if (p == 1 && filter)
      hipLaunchKernelGGL(sort_filter_kernel, dim3(256), dim3(kFilterT), 0, stream, v.jobs + kJobBig);
    if (p == kfirst) hipLaunchKernelGGL(sort_fix_kernel, dim3(nft), dim3(kT), 0, stream, v.jobs + kJobBig, p);
    hipLaunchKernelGGL(sort_hist_kernel, dim3(Jh.stride), dim3(kT), 0, stream, Jh, p);
    hipLaunchKernelGGL(sort_scan_kernel, dim3(256), dim3(kT), 0, stream, Jb, p);
    hipLaunchKernelGGL(sort_scatter_kernel, dim3(nt), dim3(kST), 0, stream, Jb, p);
  }
  // Pairing and the pair list.
  PairArgs P;
  P.ev = events;
  P.ad_job = v.jobs + kJobAd;
  P.n_ad = &ctl->n_ad;
  P.ad_idx = v.S.ad_idx;
  P.ad_op = v.S.ad_op;
  P.ad_w_dev = v.S.ad_w_dev;
  P.ad_w_addr = v.S.ad_w_addr;
  P.ad_alloc_partner = v.S.ad_alloc_partner;
  P.tile_cnt = v.tile_cnt;
  P.pr_alloc = v.pr_alloc;
  P.pr_del = v.pr_del;
  P.pr_w_bytes = v.pr_w_bytes;
  P.pr_w_dev = v.pr_w_dev;
  P.pr_w_haddr = v.pr_w_haddr;
  P.flags = out_flags;
  P.ctl = ctl;
  P.rep = out_report;
  // Beside them the duplicates and round trips, on the caller's stream.
  DDArgs D;
  D.ev = events;
  D.n = nn;
  D.aux = v.aux;
  D.job = v.jobs + kJobBig;
  D.ctl = ctl;
  D.agg = v.agg;
  D.carry = v.carry;
  D.flags = out_flags;
  D.rep = out_report;
  D.parts = v.parts;
  D.uth = nullptr;
  hipLaunchKernelGGL(sort_fix_kernel, dim3(nft), dim3(kT), 0, stream, v.jobs + kJobBig, kFixFinal);
  hipLaunchKernelGGL(pair_kernel, dim3(grid_map), dim3(kT), 0, side, P);
  hipLaunchKernelGGL(ddrt_agg_kernel<kRounds>, dim3(nt), dim3(kT), 0, stream, D);
  hipLaunchKernelGGL(pair_count_kernel, dim3(nt), dim3(kT), 0, side, P);
  hipLaunchKernelGGL(ddrt_carry_kernel, dim3(1), dim3(kCT), 0, stream, D, nt * (kT / 64));
  hipLaunchKernelGGL(scan_counts_kernel<2>, dim3(1), dim3(1024), 0, side, v.tile_cnt, nt, &ctl->n_pairs, nullptr);
  hipLaunchKernelGGL((ddrt_final_kernel<kRounds, false>), dim3(nt), dim3(kT), 0, stream, D);
  hipLaunchKernelGGL(pair_scatter_kernel, dim3(nt), dim3(kT), 0, side, P);
  hipLaunchKernelGGL(reduce_parts_kernel, dim3(S_ELIM_TX + 1 - S_DD_EVENTS), dim3(kT), 0, stream, v.parts, nt,
                     (uint32_t)S_DD_EVENTS, ctl, out_report, plan_none);
  const KernRangeArgs K{v.jobs + kJobKs, v.jobs + kJobKe, v.S.k_w_dev, v.S.k_w_start, v.S.k_w_end,
                        &ctl->n_k, v.starts_sorted, v.ends_sorted, ctl};
  hipLaunchKernelGGL(side_misc_kernel, dim3(grid_map), dim3(kT), 0, side, K, U, v.pt, &ctl->n_pairs);
  hipLaunchKernelGGL(ut_eval_kernel, dim3(grid_map), dim3(kT), 0, side, U);

  // Pairs grouped by (host address, device, bytes) in a table (cleared above).
  hipLaunchKernelGGL(pair_table_insert_kernel, dim3(grid_pair), dim3(kT), 0, side, v.pt, &ctl->n_pairs,
                     v.pr_w_haddr, v.pr_w_dev, v.pr_w_bytes);

  RaArgs R;
  R.ev = events;
  R.T = v.pt;
  R.starts_sorted = v.starts_sorted;
  R.ends_sorted = v.ends_sorted;
  R.n_pairs = &ctl->n_pairs;
  R.pr_alloc = v.pr_alloc;
  R.pr_del = v.pr_del;
  R.ad_idx = v.S.ad_idx;
  R.pr_w_bytes = v.pr_w_bytes;
  R.pr_w_dev = v.pr_w_dev;
  R.pr_w_haddr = v.pr_w_haddr;
  R.ad_kc = v.S.ad_kc;
  R.ad_km = v.S.ad_km;
  R.kd_ts = v.S.kd_ts;
  R.ctl = ctl;
  R.flags = out_flags;
  R.parts = v.parts;
  hipLaunchKernelGGL(ra_ua_kernel, dim3(grid_sum), dim3(kT), 0, side, R);
  hipLaunchKernelGGL(reduce_parts_kernel, dim3(S_ELIM_PAIRS + 1 - S_RA_EVENTS), dim3(kT), 0, side, v.parts, grid_sum,
                     (uint32_t)S_RA_EVENTS, ctl, out_report, plan_none);
  if (alg2_rx) {
    Alg2Args G;
    G.job = v.jobs + kJobBig;
    G.aux = v.aux;
    G.n = nn;
    G.rx = alg2_rx;
    G.npairs = alg2_np;
    hipLaunchKernelGGL(alg2_kernel, dim3(ceil_div32(n, kT)), dim3(kT), 0, stream, G);
  }

  ODP_HIP(hipEventRecord(ws->a_join, side));

  ODP_HIP(hipStreamWaitEvent(stream, ws->a_join, 0));
  hipLaunchKernelGGL(ut_merge_kernel, dim3(grid_sum), dim3(kT), 0, stream, U);
  hipLaunchKernelGGL(finalize_kernel, dim3(1), dim3(kT), 0, stream, v.parts, grid_sum, ctl, out_report);
  return check_hip(hipGetLastError(), "odp_analyze_trace launch");
}

// The analysis of kTinyMax < n <= kWalkMax records, in arrays of the same workspace.
static int enqueue_walks(Workspace* ws, const odp_event* events, size_t n, uint8_t* out_flags, odp_report* out_report,
                         hipStream_t stream) {
  const Views v = views(ws);
  WalkArgs A;
  A.ev = events;
  A.n = (uint32_t)n;
  A.flags = out_flags;
  A.rep = out_report;
  A.pair = v.bv[0];
  A.sums = v.skey[0];
  A.ctl = v.ctl;
  const uint32_t blocks = ceil_div32(n, kWalkRec), pblocks = ceil_div32(n, kWalkPairRec);
  // (the workspace holds at least 4,096 records with 2 * kSubsetJobs sort key words each)
  static_assert((kWalkMax / kWalkRec + kWalkMax / kWalkPairRec) * kWalkAcc <= 2 * kSubsetJobs * 4096, "sums fit the sort keys");
  hipLaunchKernelGGL(walk_kernel, dim3(blocks), dim3(kWalkT), 0, stream, A);
  hipLaunchKernelGGL(walk_pairs_kernel, dim3(pblocks), dim3(kWalkT), 0, stream, A, blocks);
  return check_hip(hipGetLastError(), "odp_analyze_trace launch");
}

extern "C" int odp_analyze_trace(const odp_event* events, size_t n, uint8_t* out_flags, odp_report* out_report,
                                 odp_stream_t stream_) {
  hipStream_t stream = static_cast<hipStream_t>(stream_);
  if (n > 0xFFFFFFFFull) return set_error(ODP_ERANGE, "odp_analyze_trace: n = %zu above 2^32 - 1", n);
  if (!out_report) return set_error(ODP_EINVAL, "odp_analyze_trace: null report");
  if (n > 0 && (!events || !out_flags)) return set_error(ODP_EINVAL, "odp_analyze_trace: null array with n = %zu", n);
  if (n <= kTinyMax) {
    // one workgroup, no workspace
    hipLaunchKernelGGL(analyze_tiny_kernel, dim3(1), dim3(kTinyMax), 0, stream, events, (uint32_t)n, out_flags,
                       out_report);
    return check_hip(hipGetLastError(), "odp_analyze_trace launch");
  }
  int err = 0;
  Workspace* ws = workspace_for(stream, &err);
  if (!ws) return err;
  hipStreamCaptureStatus capst = hipStreamCaptureStatusNone;
  ODP_HIP(hipStreamIsCapturing(stream, &capst));
  const bool capturing = capst != hipStreamCaptureStatusNone;
  if (n > ws->a_cap_events || !ws->a_cap_events) {
    if (capturing)
      return set_error(ODP_ENOMEM, "odp_analyze_trace: workspace for %zu records not reserved before capture", n);
    int e = analyze_reserve(ws, n);
    if (e) return e;
  }
  if (n <= kWalkMax) return enqueue_walks(ws, events, n, out_flags, out_report, stream);
  if (capturing) return enqueue_analysis(ws, events, n, out_flags, out_report, stream);
  // The sequence is 13 or 76 launches on two streams; a call repeated with the
  // same arguments replays it as one graph instead (the first repeat captures
  // it), so the host's launch cost leaves the device's time.
  const bool same = ws->ag_ev == events && ws->ag_n == n && ws->ag_flags == out_flags && ws->ag_rep == out_report;
  if (!same) {
    if (ws->a_graph) {
      ODP_HIP(hipGraphExecDestroy(ws->a_graph));
      ws->a_graph = nullptr;
    }
    ws->ag_ev = events;
    ws->ag_n = n;
    ws->ag_flags = out_flags;
    ws->ag_rep = out_report;
    return enqueue_analysis(ws, events, n, out_flags, out_report, stream);
  }
  if (!ws->a_graph) {
    hipStream_t cs;
    ODP_HIP(hipStreamCreateWithFlags(&cs, hipStreamNonBlocking));
    hipGraph_t g = nullptr;
    hipError_t he = hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal);
    int e = ODP_OK;
    if (he == hipSuccess) {
      e = enqueue_analysis(ws, events, n, out_flags, out_report, cs);
      he = hipStreamEndCapture(cs, &g);
    }
    (void)hipStreamDestroy(cs);
    if (he != hipSuccess) return check_hip(he, "analysis graph capture");
    if (e) {
      if (g) (void)hipGraphDestroy(g);
      return e;
    }
    he = hipGraphInstantiate(&ws->a_graph, g, nullptr, nullptr, 0);
    (void)hipGraphDestroy(g);
    if (he != hipSuccess) {
      ws->a_graph = nullptr;
      return check_hip(he, "analysis graph instantiate");
    }
  }
  ODP_HIP(hipGraphLaunch(ws->a_graph, stream));
  return ODP_OK;
}

extern "C" int odp_analyze_trace_alg2(const odp_event* events, size_t n, uint8_t* out_flags, odp_report* out_report,
                                      uint32_t* out_rx, uint64_t* out_npairs, odp_stream_t stream_) {
  hipStream_t stream = static_cast<hipStream_t>(stream_);
  if (n > 0xFFFFFFFFull) return set_error(ODP_ERANGE, "odp_analyze_trace_alg2: n = %zu above 2^32 - 1", n);
  if (!out_report || !out_npairs) return set_error(ODP_EINVAL, "odp_analyze_trace_alg2: null report or pair count");
  if (n > 0 && (!events || !out_flags || !out_rx))
    return set_error(ODP_EINVAL, "odp_analyze_trace_alg2: null array with n = %zu", n);
  int err = 0;
  Workspace* ws = workspace_for(stream, &err);
  if (!ws) return err;
  hipStreamCaptureStatus capst = hipStreamCaptureStatusNone;
  ODP_HIP(hipStreamIsCapturing(stream, &capst));
  if (n > ws->a_cap_events || !ws->a_cap_events) {
    if (capst != hipStreamCaptureStatusNone)
      return set_error(ODP_ENOMEM, "odp_analyze_trace_alg2: workspace for %zu records not reserved before capture", n);
    int e = analyze_reserve(ws, n);
    if (e) return e;
  }
  return enqueue_analysis(ws, events, n, out_flags, out_report, stream, out_rx,
                          reinterpret_cast<unsigned long long*>(out_npairs));
}
