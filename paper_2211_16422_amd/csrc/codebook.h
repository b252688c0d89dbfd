// Host-side generation of the position and level hypervector tables.
#pragma once
#include <stdint.h>

#include <vector>

namespace homs {

// The flip orders of the ID_LEVEL tables: row i of the position table is row 0
// with the components id_order[0 .. floor(alpha i / (f - 1))) flipped, row j of
// the level table is row 0 with level_order[0 .. floor((D / 2) j / (Q - 1)))
// flipped. Empty for the other encodings.
struct CodebookOrders {
    std::vector<uint32_t> id_order, level_order;
};

// id_table: f rows of D/32 words; level_table: Q rows of D/32 words.
// Requires D % 64 == 0, f >= 1, Q >= 2, alpha <= D.
// encoding: HOMS_ENCODING_* (random position rows unless ID_LEVEL)
void generate_codebook(uint32_t D, uint32_t f, uint32_t Q, uint32_t alpha, uint64_t seed,
                       uint32_t encoding, uint32_t* id_table, uint32_t* level_table,
                       CodebookOrders* orders = nullptr);

// Components grouped for the step-function encoding (encode.hip states it).
// Component d has the class 2 (u - 1) + c0: u the first level that flips it
// (Q when none does), c0 = bit d of F_0 xor bit d of L_0. A class's slots are
// its position-flipped components in flip order, then one slot for all its
// other components.
struct EncodeClasses {
    uint32_t classes = 0;             // 2 Q
    uint32_t slots = 0;               // over all classes
    std::vector<uint32_t> start;      // [classes] first slot of each class
    std::vector<uint16_t> source;     // [D] slot of each component
    std::vector<uint16_t> first_off;  // [alpha + 1][classes] slot of the class's first component
                                      // whose flip rank is at least K
};
EncodeClasses make_encode_classes(uint32_t D, uint32_t Q, uint32_t alpha, const uint32_t* id_row0,
                                  const uint32_t* level_row0, const CodebookOrders& orders);

}  // namespace homs
