// Wide chains and sweeps: H of 1537 - 2048.
#include "resident_wide.h"

namespace mebptt {

Table<WideConfig> wide_table_2() {
  static const WideConfig table[] = {
      wide_config_of<WideKind<4, 16, 0, 0, 0, 4, 0, 0, 1>>(),
      wide_config_of<WideKind<4, 16, 0, 0, 0, 4, 0, 0, 2>>(),
      wide_config_of<WideKind<4, 16, 1, 0, 0, 4, 3, 0, 4>>(),
  };
  return {table, (int)(sizeof table / sizeof table[0])};
}

}  // namespace mebptt
