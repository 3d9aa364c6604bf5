// Wide chains and sweeps: H of 2049 - 4096.
#include "resident_wide.h"

namespace mebptt {

Table<WideConfig> wide_table_3() {
  static const WideConfig table[] = {
      wide_config_of<WideKind<3, 24, 0, 0, 0, 6, 0, 0, 1>>(),
      wide_config_of<WideKind<3, 24, 0, 0, 0, 6, 0, 0, 2>>(),
      wide_config_of<WideKind<4, 32, 7, 4, 0, 0, 7, 6, 1>>(),
      wide_config_of<WideKind<4, 32, 7, 4, 0, 0, 7, 6, 2>>(),
  };
  return {table, (int)(sizeof table / sizeof table[0])};
}

}  // namespace mebptt
