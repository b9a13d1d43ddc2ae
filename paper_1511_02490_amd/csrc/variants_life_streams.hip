// Variants: Game of Life in registers.
#include "variants.h"

void register_life_streams(std::vector<Variant> &r) {
    reg_life_stream(r, 4);
    reg_life_stream(r, 8);
    reg_life_stream(r, 16);
}
