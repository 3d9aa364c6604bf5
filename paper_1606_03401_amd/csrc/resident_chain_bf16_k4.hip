// Forward chains, bf16 operands, at most 20 macro steps of K (KX + KH <= 640): K split over 4 waves.
#include "resident.h"

namespace mebptt {

Table<ChainConfig> chain_table_bf16_k4() {
  static const ChainConfig table[] = {
      MEBPTT_CHAIN(__bf16, 1, 1, 0, 1, 4, 0),
      MEBPTT_CHAIN(__bf16, 1, 1, 0, 1, 4, 1),
      MEBPTT_CHAIN(__bf16, 1, 1, 0, 1, 4, 2),
      MEBPTT_CHAIN(__bf16, 1, 2, 0, 1, 4, 0),
      MEBPTT_CHAIN(__bf16, 1, 2, 0, 1, 4, 1),
      MEBPTT_CHAIN(__bf16, 1, 2, 0, 1, 4, 2),
      MEBPTT_CHAIN(__bf16, 1, 5, 0, 1, 4, 0),
      MEBPTT_CHAIN(__bf16, 1, 5, 0, 1, 4, 1),
      MEBPTT_CHAIN(__bf16, 1, 5, 0, 1, 4, 2),
      MEBPTT_CHAIN(__bf16, 2, 2, 0, 2, 4, 0),
      MEBPTT_CHAIN(__bf16, 2, 2, 0, 2, 4, 1),
      MEBPTT_CHAIN(__bf16, 2, 2, 0, 2, 4, 2),
      MEBPTT_CHAIN(__bf16, 2, 4, 0, 2, 4, 0),
      MEBPTT_CHAIN(__bf16, 2, 4, 0, 2, 4, 1),
      MEBPTT_CHAIN(__bf16, 2, 4, 0, 2, 4, 2),
      MEBPTT_CHAIN(__bf16, 3, 3, 0, 3, 4, 0),
      MEBPTT_CHAIN(__bf16, 3, 3, 0, 3, 4, 1),
      MEBPTT_CHAIN(__bf16, 3, 3, 0, 3, 4, 2),
      MEBPTT_CHAIN(__bf16, 4, 1, 0, 4, 4, 0),
      MEBPTT_CHAIN(__bf16, 4, 1, 0, 4, 4, 1),
      MEBPTT_CHAIN(__bf16, 4, 1, 0, 4, 4, 2),
      MEBPTT_CHAIN(__bf16, 4, 2, 0, 4, 4, 0),
      MEBPTT_CHAIN(__bf16, 4, 2, 0, 4, 4, 1),
      MEBPTT_CHAIN(__bf16, 4, 2, 0, 4, 4, 2),
      MEBPTT_CHAIN(__bf16, 5, 1, 0, 5, 4, 0),
      MEBPTT_CHAIN(__bf16, 5, 1, 0, 5, 4, 1),
      MEBPTT_CHAIN(__bf16, 5, 1, 0, 5, 4, 2),
  };
  return {table, (int)(sizeof table / sizeof table[0])};
}

}  // namespace mebptt
