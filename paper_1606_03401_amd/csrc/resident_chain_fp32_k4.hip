// Forward chains, fp32 operands, at most 20 macro steps of K (KX + KH <= 320): K split over 4 waves.
#include "resident.h"

namespace mebptt {

Table<ChainConfig> chain_table_fp32_k4() {
  static const ChainConfig table[] = {
      MEBPTT_CHAIN(float, 1, 2, 0, 2, 4, 0),
      MEBPTT_CHAIN(float, 1, 2, 0, 2, 4, 1),
      MEBPTT_CHAIN(float, 1, 2, 0, 2, 4, 2),
      MEBPTT_CHAIN(float, 1, 5, 0, 2, 4, 0),
      MEBPTT_CHAIN(float, 1, 5, 0, 2, 4, 1),
      MEBPTT_CHAIN(float, 1, 5, 0, 2, 4, 2),
      MEBPTT_CHAIN(float, 2, 3, 0, 4, 4, 0),
      MEBPTT_CHAIN(float, 2, 3, 0, 4, 4, 1),
      MEBPTT_CHAIN(float, 2, 3, 0, 4, 4, 2),
      MEBPTT_CHAIN(float, 3, 1, 0, 5, 4, 0),
      MEBPTT_CHAIN(float, 3, 1, 0, 5, 4, 1),
      MEBPTT_CHAIN(float, 3, 1, 0, 5, 4, 2),
  };
  return {table, (int)(sizeof table / sizeof table[0])};
}

}  // namespace mebptt
