// Forward chains, bf16 operands, more than 20 macro steps of K: K split over 8 waves.
#include "resident.h"

namespace mebptt {

Table<ChainConfig> chain_table_bf16_k8() {
  static const ChainConfig table[] = {
      MEBPTT_CHAIN(__bf16, 1, 4, 0, 1, 8, 0),
      MEBPTT_CHAIN(__bf16, 1, 4, 0, 1, 8, 1),
      MEBPTT_CHAIN(__bf16, 1, 4, 0, 1, 8, 2),
      MEBPTT_CHAIN(__bf16, 1, 8, 0, 1, 8, 0),
      MEBPTT_CHAIN(__bf16, 1, 8, 0, 1, 8, 1),
      MEBPTT_CHAIN(__bf16, 1, 8, 0, 1, 8, 2),
      MEBPTT_CHAIN(__bf16, 2, 4, 0, 1, 8, 0),
      MEBPTT_CHAIN(__bf16, 2, 4, 0, 1, 8, 1),
      MEBPTT_CHAIN(__bf16, 2, 4, 0, 1, 8, 2),
      MEBPTT_CHAIN(__bf16, 3, 4, 0, 2, 8, 0),
      MEBPTT_CHAIN(__bf16, 3, 4, 0, 2, 8, 1),
      MEBPTT_CHAIN(__bf16, 3, 4, 0, 2, 8, 2),
      MEBPTT_CHAIN(__bf16, 4, 2, 0, 2, 8, 0),
      MEBPTT_CHAIN(__bf16, 4, 2, 0, 2, 8, 1),
      MEBPTT_CHAIN(__bf16, 4, 2, 0, 2, 8, 2),
      MEBPTT_CHAIN(__bf16, 4, 4, 0, 2, 8, 0),
      MEBPTT_CHAIN(__bf16, 4, 4, 0, 2, 8, 1),
      MEBPTT_CHAIN(__bf16, 4, 4, 0, 2, 8, 2),
      MEBPTT_CHAIN(__bf16, 5, 2, 0, 3, 8, 0),
      MEBPTT_CHAIN(__bf16, 5, 2, 0, 3, 8, 1),
      MEBPTT_CHAIN(__bf16, 5, 4, 0, 3, 8, 0),
      MEBPTT_CHAIN(__bf16, 5, 4, 0, 3, 8, 1),
      MEBPTT_CHAIN(__bf16, 6, 2, 0, 3, 8, 0),
      MEBPTT_CHAIN(__bf16, 6, 2, 0, 3, 8, 1),
      MEBPTT_CHAIN(__bf16, 6, 3, 1, 3, 8, 0),
      MEBPTT_CHAIN(__bf16, 6, 3, 1, 3, 8, 1),
      MEBPTT_CHAIN(__bf16, 6, 4, 2, 3, 8, 0),
      MEBPTT_CHAIN(__bf16, 6, 4, 2, 3, 8, 1),
      MEBPTT_CHAIN(__bf16, 7, 1, 1, 4, 8, 0),
      MEBPTT_CHAIN(__bf16, 7, 1, 1, 4, 8, 1),
      MEBPTT_CHAIN(__bf16, 7, 2, 1, 4, 8, 0),
      MEBPTT_CHAIN(__bf16, 7, 2, 1, 4, 8, 1),
      MEBPTT_CHAIN(__bf16, 8, 1, 1, 4, 8, 0),
      MEBPTT_CHAIN(__bf16, 8, 1, 1, 4, 8, 1),
  };
  return {table, (int)(sizeof table / sizeof table[0])};
}

}  // namespace mebptt
