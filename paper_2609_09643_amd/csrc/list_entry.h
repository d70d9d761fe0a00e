// list_entry.h -- the words and sizes of the sorted-list pool (lane.hip), for
// host and device code.
#pragma once

#include <cstdint>

namespace unison {

constexpr uint32_t kListSlotBits = 12;
constexpr uint32_t kListResidents = 1u << kListSlotBits;

// A resident as one word, session << 12 | slot: 20 + 12 bits, every value of
// which is an entry (the largest session in the last slot is 0xFFFFFFFF).
constexpr uint32_t list_word(uint32_t sid, uint32_t slot) { return (sid << kListSlotBits) | slot; }
constexpr uint32_t list_sid(uint32_t w) { return w >> kListSlotBits; }
constexpr uint32_t list_slot(uint32_t w) { return w & (kListResidents - 1u); }

// Which list the next fired timer is in (1: SRAM), by each list's leaves with a
// fired entry and its smallest fired word: the word of an empty choice is
// 0xFFFFFFFF, which may also be an entry's, so the leaves tell whether there is one.
constexpr uint32_t fired_in_sram(uint32_t hbm_leaves, uint32_t sram_leaves, uint32_t hbm, uint32_t sram) {
  return (sram_leaves != 0u) & ((hbm_leaves == 0u) | (sram < hbm)) ? 1u : 0u;
}

// Rows for the leaves of max_res residents.  Packed, both lists use a row per 64
// residents and one more: a third of them or less up to 3,072 residents, 65 of the
// 152 that LDS has beside the slots at 4,096.
constexpr uint32_t list_rows(uint64_t max_res) {
  const uint32_t full = (uint32_t)((max_res + 63) / 64);
  return 3u * full + 8u < 152u ? 3u * full + 8u : 152u;
}
// An insertion takes at most one row, so any row free after packing is enough; so
// many keep the packing rare.
static_assert(list_rows(kListResidents) - (kListResidents / 64u + 1u) >= kListResidents / 64u,
              "packed leaves leave as many rows free as they fill");

}  // namespace unison
