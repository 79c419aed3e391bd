// Occupancy caps by dynamic LDS: a streaming launch reserves LDS that nothing
// uses, so that no more than a chosen number of its blocks run on a CU.
#pragma once

namespace edit {

// A CU hands out LDS in pieces of this size: counted with blocks that wait for
// each other, 26,880 bytes let six run on a CU and 26,881 five, 20,480 eight
// and 20,481 seven (the runtime's occupancy query, which does not round up,
// says six at 27,136 bytes and five at 32,768, where five and four run).
constexpr int kLdsPiece = 1280;
constexpr int kLdsPerCu = 160 * 1024;

// Blocks of `lds` bytes, static and dynamic, that a CU holds.
constexpr int lds_blocks(int lds, int lds_per_cu) {
  return lds_per_cu / kLdsPiece / ((lds + kLdsPiece - 1) / kLdsPiece);
}

// The most dynamic LDS that lets `blocks` blocks of a kernel with
// `static_lds` bytes of its own run on a CU.
constexpr int lds_for_blocks(int blocks, int static_lds, int lds_per_cu) {
  const int lds = lds_per_cu / kLdsPiece / blocks * kLdsPiece - static_lds;
  return lds > 0 ? lds : 0;
}

}  // namespace edit
