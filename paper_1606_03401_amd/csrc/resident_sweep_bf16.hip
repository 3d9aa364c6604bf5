// Sweeps with forward operations, bf16 operands.
#include "resident_sweep.h"

namespace mebptt {

Table<SweepConfig> sweep_table_bf16() {
  static const SweepConfig table[] = {
      MEBPTT_SWEEP(__bf16, 1, 1, 1, 4, 4, 0, 4, 0),
      MEBPTT_SWEEP(__bf16, 1, 1, 1, 4, 4, 0, 4, 1),
      MEBPTT_SWEEP(__bf16, 1, 1, 1, 4, 4, 0, 4, 2),
      MEBPTT_SWEEP(__bf16, 1, 2, 1, 4, 4, 0, 4, 0),
      MEBPTT_SWEEP(__bf16, 1, 2, 1, 4, 4, 0, 4, 1),
      MEBPTT_SWEEP(__bf16, 1, 2, 1, 4, 4, 0, 4, 2),
      MEBPTT_SWEEP(__bf16, 1, 5, 1, 4, 4, 0, 4, 0),
      MEBPTT_SWEEP(__bf16, 1, 5, 1, 4, 4, 0, 4, 1),
      MEBPTT_SWEEP(__bf16, 1, 5, 1, 4, 4, 0, 4, 2),
      MEBPTT_SWEEP(__bf16, 2, 2, 2, 4, 4, 0, 8, 0),
      MEBPTT_SWEEP(__bf16, 2, 2, 2, 4, 4, 0, 8, 1),
      MEBPTT_SWEEP(__bf16, 2, 2, 2, 4, 4, 0, 8, 2),
      MEBPTT_SWEEP(__bf16, 2, 4, 2, 4, 4, 0, 8, 0),
      MEBPTT_SWEEP(__bf16, 2, 4, 2, 4, 4, 0, 8, 1),
      MEBPTT_SWEEP(__bf16, 2, 4, 2, 4, 4, 0, 8, 2),
      MEBPTT_SWEEP(__bf16, 3, 3, 3, 4, 6, 0, 8, 0),
      MEBPTT_SWEEP(__bf16, 3, 3, 3, 4, 6, 0, 8, 1),
      MEBPTT_SWEEP(__bf16, 3, 3, 3, 4, 6, 6, 8, 2),
      MEBPTT_SWEEP(__bf16, 4, 1, 4, 4, 8, 0, 8, 0),
      MEBPTT_SWEEP(__bf16, 4, 1, 4, 4, 8, 0, 8, 1),
      MEBPTT_SWEEP(__bf16, 4, 1, 4, 4, 8, 8, 8, 2),
      MEBPTT_SWEEP(__bf16, 4, 2, 4, 4, 8, 0, 8, 0),
      MEBPTT_SWEEP(__bf16, 4, 2, 4, 4, 8, 0, 8, 1),
      MEBPTT_SWEEP(__bf16, 1, 4, 1, 8, 4, 0, 4, 0),
      MEBPTT_SWEEP(__bf16, 1, 4, 1, 8, 4, 0, 4, 1),
      MEBPTT_SWEEP(__bf16, 1, 4, 1, 8, 4, 0, 4, 2),
      MEBPTT_SWEEP(__bf16, 1, 8, 1, 8, 4, 0, 4, 0),
      MEBPTT_SWEEP(__bf16, 1, 8, 1, 8, 4, 0, 4, 1),
      MEBPTT_SWEEP(__bf16, 2, 4, 1, 8, 4, 0, 8, 0),
      MEBPTT_SWEEP(__bf16, 2, 4, 1, 8, 4, 0, 8, 1),
      MEBPTT_SWEEP(__bf16, 2, 4, 1, 8, 4, 0, 8, 2),
      MEBPTT_SWEEP(__bf16, 3, 4, 2, 8, 6, 0, 8, 0),
      MEBPTT_SWEEP(__bf16, 3, 4, 2, 8, 6, 0, 8, 1),
      MEBPTT_SWEEP(__bf16, 4, 4, 2, 8, 8, 8, 8, 0),
      MEBPTT_SWEEP(__bf16, 4, 4, 2, 8, 8, 8, 8, 1),
  };
  return {table, (int)(sizeof table / sizeof table[0])};
}

}  // namespace mebptt
