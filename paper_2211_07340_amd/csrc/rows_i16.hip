// The row-lane kernel on int16 references (see rows.h).
#include "rows.h"

namespace sdtw {
hipError_t launch_rows_i16(const RowsArgs& a, hipStream_t st, int parts) {
  return launch_rows<FmtI16, false>(a, st, parts);
}
}  // namespace sdtw
