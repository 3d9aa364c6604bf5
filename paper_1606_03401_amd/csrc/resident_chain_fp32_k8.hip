// Forward chains, fp32 operands, more than 20 macro steps of K: K split over 8 waves.
#include "resident.h"

namespace mebptt {

Table<ChainConfig> chain_table_fp32_k8() {
  static const ChainConfig table[] = {
      MEBPTT_CHAIN(float, 1, 4, 0, 1, 8, 0),
      MEBPTT_CHAIN(float, 1, 4, 0, 1, 8, 1),
      MEBPTT_CHAIN(float, 1, 4, 0, 1, 8, 2),
      MEBPTT_CHAIN(float, 1, 8, 0, 1, 8, 0),
      MEBPTT_CHAIN(float, 1, 8, 0, 1, 8, 1),
      MEBPTT_CHAIN(float, 1, 8, 0, 1, 8, 2),
      MEBPTT_CHAIN(float, 2, 2, 0, 2, 8, 0),
      MEBPTT_CHAIN(float, 2, 2, 0, 2, 8, 1),
      MEBPTT_CHAIN(float, 2, 2, 0, 2, 8, 2),
      MEBPTT_CHAIN(float, 2, 4, 0, 2, 8, 0),
      MEBPTT_CHAIN(float, 2, 4, 0, 2, 8, 1),
      MEBPTT_CHAIN(float, 2, 4, 0, 2, 8, 2),
      MEBPTT_CHAIN(float, 2, 8, 0, 2, 8, 0),
      MEBPTT_CHAIN(float, 2, 8, 0, 2, 8, 1),
      MEBPTT_CHAIN(float, 2, 8, 0, 2, 8, 2),
      MEBPTT_CHAIN(float, 3, 4, 0, 3, 8, 0),
      MEBPTT_CHAIN(float, 3, 4, 0, 3, 8, 1),
      MEBPTT_CHAIN(float, 3, 4, 0, 3, 8, 2),
      MEBPTT_CHAIN(float, 4, 2, 0, 4, 8, 0),
      MEBPTT_CHAIN(float, 4, 2, 0, 4, 8, 1),
      MEBPTT_CHAIN(float, 4, 2, 0, 4, 8, 2),
      MEBPTT_CHAIN(float, 4, 4, 0, 4, 8, 0),
      MEBPTT_CHAIN(float, 4, 4, 0, 4, 8, 1),
      MEBPTT_CHAIN(float, 4, 4, 2, 4, 8, 2),
      MEBPTT_CHAIN(float, 4, 8, 3, 4, 8, 0),
      MEBPTT_CHAIN(float, 4, 8, 3, 4, 8, 1),
  };
  return {table, (int)(sizeof table / sizeof table[0])};
}

}  // namespace mebptt
