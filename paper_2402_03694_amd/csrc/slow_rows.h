// Slow model, register form (slow_rows.hip): the tile form's arguments and what follows from them.
#pragma once

#include "slow_tiles.h"

namespace sfrows {

struct RowsArgs : sftiles::FusedArgs {
    float clamp_z;     // the input map's clamp, infinity without a map
    uint32_t nb1, nb2; // column blocks of the hidden layers
    uint32_t ks2, ks3; // k-steps of the second and third layer as their weights are ordered
};

// For models the tile form takes, with 16-byte aligned input rows of at most 128 values, a multiple of 4
int run(sf_ctx* ctx, const RowsArgs& a);

} // namespace sfrows
