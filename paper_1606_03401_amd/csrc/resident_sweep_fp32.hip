// Sweeps, fp32 operands.
#include "resident_sweep.h"

namespace mebptt {

Table<SweepConfig> sweep_table_fp32() {
  static const SweepConfig table[] = {
      MEBPTT_SWEEP(float, 1, 2, 2, 4, 4, 0, 4, 1),
      MEBPTT_SWEEP(float, 1, 2, 2, 4, 4, 0, 4, 2),
      MEBPTT_SWEEP(float, 1, 5, 2, 4, 4, 0, 4, 1),
      MEBPTT_SWEEP(float, 1, 5, 2, 4, 4, 0, 4, 2),
      MEBPTT_SWEEP(float, 1, 2, 2, 4, 4, 0, 8, 1),
      MEBPTT_SWEEP(float, 1, 2, 2, 4, 4, 0, 8, 2),
      MEBPTT_SWEEP(float, 1, 5, 2, 4, 4, 0, 8, 1),
      MEBPTT_SWEEP(float, 1, 5, 2, 4, 4, 0, 8, 2),
      MEBPTT_SWEEP(float, 2, 3, 4, 4, 8, 0, 8, 1),
      MEBPTT_SWEEP(float, 1, 4, 1, 8, 4, 0, 4, 1),
      MEBPTT_SWEEP(float, 1, 4, 1, 8, 4, 0, 4, 2),
      MEBPTT_SWEEP(float, 1, 8, 1, 8, 4, 0, 4, 1),
      MEBPTT_SWEEP(float, 1, 4, 1, 8, 4, 0, 8, 1),
      MEBPTT_SWEEP(float, 1, 4, 1, 8, 4, 0, 8, 2),
      MEBPTT_SWEEP(float, 1, 8, 1, 8, 4, 0, 8, 1),
      MEBPTT_SWEEP(float, 2, 2, 2, 8, 8, 0, 8, 1),
      MEBPTT_SWEEP(float, 2, 4, 2, 8, 8, 0, 8, 1),
  };
  return {table, (int)(sizeof table / sizeof table[0])};
}

Table<BackSweepConfig> back_sweep_table_fp32() {
  static const BackSweepConfig table[] = {
      MEBPTT_BACK_SWEEP(float, 1, 4, 0, 4, 0),
      MEBPTT_BACK_SWEEP(float, 1, 4, 0, 4, 1),
      MEBPTT_BACK_SWEEP(float, 1, 4, 0, 4, 2),
      MEBPTT_BACK_SWEEP(float, 1, 4, 0, 8, 0),
      MEBPTT_BACK_SWEEP(float, 1, 4, 0, 8, 1),
      MEBPTT_BACK_SWEEP(float, 1, 4, 0, 8, 2),
      MEBPTT_BACK_SWEEP(float, 2, 8, 0, 8, 0),
      MEBPTT_BACK_SWEEP(float, 2, 8, 0, 8, 1),
      MEBPTT_BACK_SWEEP(float, 2, 8, 0, 8, 2),
      MEBPTT_BACK_SWEEP(float, 3, 12, 0, 8, 0),
      MEBPTT_BACK_SWEEP(float, 3, 12, 0, 8, 1),
      MEBPTT_BACK_SWEEP(float, 4, 16, 0, 8, 0),
      MEBPTT_BACK_SWEEP(float, 4, 16, 0, 8, 1),
  };
  return {table, (int)(sizeof table / sizeof table[0])};
}

}  // namespace mebptt
