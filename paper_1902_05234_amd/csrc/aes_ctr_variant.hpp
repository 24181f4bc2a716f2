// aes_ctr_variant.hpp -- choice of the CTR kernel for a piece of a host buffer
// (aes_pipe.cpp) beside that of aes_ctr_crypt (ctr_variant, aes_internal.hpp).
#pragma once
#include <cstdint>

#include "aes_internal.hpp"

namespace aesgpu {

// As ctr_variant, but with a compiled-in entry in its whole-state form
// (aes_abi.cpp).
aes_variant ctr_whole_state_variant(int nr, uint64_t nblocks);

// For a piece of nbytes bytes in the pinned staging; beside_copies: the calling
// thread copies other pieces of the buffer meanwhile (aes_pipe.cpp).
aes_variant ctr_piece_variant(int nr, uint64_t nbytes, bool beside_copies);

}  // namespace aesgpu
