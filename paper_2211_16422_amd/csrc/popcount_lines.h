// Which words the popcount tile's look-ahead touches (popcount_tile.h): one of
// each 128-byte line of the next block of library rows. Plain C++, so that the
// arithmetic can be checked on the host for every row length; constexpr
// functions are device functions too.
#pragma once
#include <stddef.h>
#include <stdint.h>

namespace homs {
namespace popc {

constexpr uint32_t kLineWords = 32;  // a 128-byte line

// 128-byte pieces of `rows` consecutive rows of `words` words (a row may be half
// a line, D = 512, or one and a half, D = 1,536: the rows count as one run)
constexpr uint32_t ahead_lines(uint32_t rows, uint32_t words)
{
    return (rows * words + kLineWords - 1) / kLineWords;
}

// the word touched in piece i of the rows from `row` on: inside them for every
// i < ahead_lines(rows, words)
constexpr size_t ahead_word(uint32_t row, uint32_t words, uint32_t i)
{
    return (size_t)row * words + (size_t)i * kLineWords;
}

}  // namespace popc
}  // namespace homs
