// Wide chains and sweeps: H of 513 - 1024 with batches of 129 - 256, H of 1025 - 1536.
#include "resident_wide.h"

namespace mebptt {

Table<WideConfig> wide_table_1() {
  static const WideConfig table[] = {
      wide_config_of<WideKind<3, 6, 0, 0, 0, 4, 0, 0, 4>>(),
      wide_config_of<WideKind<4, 8, 0, 0, 0, 4, 0, 0, 4>>(),
      wide_config_of<WideKind<3, 12, 0, 0, 4, 4, 0, 0, 1>>(),
      wide_config_of<WideKind<3, 12, 0, 0, 4, 4, 0, 0, 2>>(),
      wide_config_of<WideKind<3, 12, 0, 0, 0, 4, 0, 0, 4>>(),
  };
  return {table, (int)(sizeof table / sizeof table[0])};
}

}  // namespace mebptt
