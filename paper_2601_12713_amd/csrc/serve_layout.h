// A server's device state: its records and where each array lies in the
// server's one device block (host code only).
#pragma once
#include <cstddef>
#include <cstdint>

#include "odp.h"

namespace odp {

constexpr int kTickMax = 1024;     // records per tick (one workgroup)
// staged bytes per request: the record, the payload pointer and size, a flag
constexpr size_t kStageBytes = sizeof(odp_event) + 8 + 8 + 1;
constexpr int kDev = ODP_MAX_DEVICE + 2;  // device codes: host (-1) .. ODP_MAX_DEVICE, shifted by one
constexpr int kTables = 6;

// Open-addressing table entry; keys are three words, values two. state is
// kEmpty or the tag of the tick that claimed the slot (never kEmpty), so a
// thread tells a slot claimed earlier (keys complete and visible) from one
// another thread of its own tick is still filling in.
struct Slot {
  uint32_t state;
  uint32_t v0;
  uint64_t k0, k1, k2;
  uint64_t v1;
};

// A window waiting for its deadline (UA: an ALLOC and its DELETE; UT: a copy
// and the next copy of its place). The kernels on `dev` that meet
// [lo, deadline] are those among the first `kc` (logged before the window
// opened) whose end reaches lo, and those logged later that start by the
// deadline.
struct Pending {
  uint64_t lo, deadline;
  uint32_t id;    // the record that gets the flag
  uint32_t kc;    // kernels on dev logged before it
  uint32_t dev;   // device code (device + 1)
  uint32_t flag;  // ODP_F_UA or ODP_F_UT
};

struct ServeState {
  uint64_t last_t_start;  // t_start of the last logged record
  uint64_t n_logged;
  uint32_t overflow;      // a table ran full
  uint32_t any_invalid;   // some record was rejected: UA/UT wait for the drain
  uint32_t kcount[kDev];  // valid KERNEL records per device code
  uint32_t pend_n;        // windows waiting in pend[pend_cur]
  uint32_t pend_cur;
};

// Byte offsets in the block of a server for a log of `cap` records. The arrays
// follow each other without a gap, those of wider elements first, so `bytes`
// is what the server's budget counts and what is allocated; the last ones,
// from `zeroed` on, start at zero.
struct ServerLayout {
  uint64_t stage[2], dig[2], log, pend[2], kstart, kmaxend, link, kc_at;
  uint64_t zeroed, tables[kTables], st, known;
  uint64_t bytes;
  uint64_t table_slots;
};

inline ServerLayout server_layout(uint64_t cap) {
  ServerLayout L{};
  L.table_slots = 1024;
  while (L.table_slots < 2 * cap) L.table_slots <<= 1;
  auto place = [&](uint64_t bytes) {
    const uint64_t at = L.bytes;
    L.bytes += bytes;
    return at;
  };
  for (uint64_t& a : L.stage) a = place(kTickMax * kStageBytes);
  for (uint64_t& a : L.dig) a = place(kTickMax * 8);
  L.log = place(cap * sizeof(odp_event));
  for (uint64_t& a : L.pend) a = place(cap * sizeof(Pending));
  L.kstart = place(uint64_t(kDev) * cap * 8);
  L.kmaxend = place(uint64_t(kDev) * cap * 8);
  L.link = place(cap * 4);
  L.kc_at = place(cap * 4);
  L.zeroed = L.bytes;
  for (uint64_t& a : L.tables) a = place(L.table_slots * sizeof(Slot));
  L.st = place(sizeof(ServeState));
  L.known = place((cap + 8) & ~3ull);  // (flag bits are set in words)
  return L;
}
static_assert(kTickMax * kStageBytes % 256 == 0 && sizeof(odp_event) % 8 == 0 && sizeof(Pending) % 8 == 0 &&
                  sizeof(Slot) % 8 == 0 && sizeof(ServeState) % 8 == 0,
              "every array starts aligned to its elements");

}  // namespace odp
