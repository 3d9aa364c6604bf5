// Sweeps of backward operations only, bf16 operands.
#include "resident_sweep.h"

namespace mebptt {

Table<BackSweepConfig> back_sweep_table_bf16() {
  static const BackSweepConfig table[] = {
      MEBPTT_BACK_SWEEP(__bf16, 1, 4, 0, 4, 0),
      MEBPTT_BACK_SWEEP(__bf16, 1, 4, 0, 4, 1),
      MEBPTT_BACK_SWEEP(__bf16, 1, 4, 0, 4, 2),
      MEBPTT_BACK_SWEEP(__bf16, 2, 4, 0, 8, 0),
      MEBPTT_BACK_SWEEP(__bf16, 2, 4, 0, 8, 1),
      MEBPTT_BACK_SWEEP(__bf16, 2, 4, 0, 8, 2),
      MEBPTT_BACK_SWEEP(__bf16, 3, 6, 0, 8, 0),
      MEBPTT_BACK_SWEEP(__bf16, 3, 6, 0, 8, 1),
      MEBPTT_BACK_SWEEP(__bf16, 3, 6, 0, 8, 2),
      MEBPTT_BACK_SWEEP(__bf16, 4, 8, 0, 8, 0),
      MEBPTT_BACK_SWEEP(__bf16, 4, 8, 0, 8, 1),
      MEBPTT_BACK_SWEEP(__bf16, 4, 8, 0, 8, 2),
      MEBPTT_BACK_SWEEP(__bf16, 5, 10, 0, 8, 0),
      MEBPTT_BACK_SWEEP(__bf16, 5, 10, 0, 8, 1),
      MEBPTT_BACK_SWEEP(__bf16, 6, 12, 0, 8, 0),
      MEBPTT_BACK_SWEEP(__bf16, 6, 12, 0, 8, 1),
      MEBPTT_BACK_SWEEP(__bf16, 7, 14, 2, 8, 0),
      MEBPTT_BACK_SWEEP(__bf16, 7, 14, 2, 8, 1),
      MEBPTT_BACK_SWEEP(__bf16, 8, 16, 4, 8, 0),
      MEBPTT_BACK_SWEEP(__bf16, 8, 16, 4, 8, 1),
  };
  return {table, (int)(sizeof table / sizeof table[0])};
}

}  // namespace mebptt
