// Variants: Game of Life, several generations per launch: in registers and in local memory (whose runs of several launches are
// made in registers too).
#include "variants.h"

void register_life_streams(std::vector<Variant> &r) {
    reg_life_stream<4>(r);
    reg_life_stream<8>(r);
    reg_life_stream<16>(r);
    reg_life_temporal<1>(r);
    reg_life_temporal<2>(r);
    reg_life_temporal<4>(r);
    reg_life_temporal<8>(r);
}
