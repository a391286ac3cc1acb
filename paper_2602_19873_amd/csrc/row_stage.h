// What the rows' pass may bring into LDS of one compressed 1x1 row: plain
// arithmetic on the row's header, for host and device.
#pragma once
#include <stdint.h>

namespace sfcnl {

constexpr uint32_t kStageWords = 256;  // words of a row in LDS (longer rows are read from memory)

// Words of the row {off, cnt} to stage, given the next row's offset `next`; 0:
// none, the row is read from memory as it is decoded. A row of count 0 has no
// words of its own: build_rows records the rows that did not fit the pool so,
// with the offsets they would have had, beyond its end. A length below the
// two bitmask words of every 64 neighbours is not this row's.
constexpr uint32_t row_stage_words(uint32_t off, uint32_t cnt, uint32_t next) {
    const uint32_t len = next - off;
    return cnt != 0u && len <= kStageWords && len >= 2u * (cnt / 64u + (cnt % 64u != 0u)) ? len : 0u;
}

}  // namespace sfcnl
