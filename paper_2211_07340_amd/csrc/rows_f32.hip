// The row-lane kernel on float32 references (see rows.h).
#include "rows.h"

namespace sdtw {
hipError_t launch_rows_f32(const RowsArgs& a, hipStream_t st, int parts) {
  return launch_rows<FmtF32, false>(a, st, parts);
}
}  // namespace sdtw
