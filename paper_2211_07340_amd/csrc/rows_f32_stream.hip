// The row-lane kernel on float32 references, extending resident rows (see rows.h).
#include "rows.h"

namespace sdtw {
hipError_t launch_rows_f32_stream(const RowsArgs& a, hipStream_t st, int parts) {
  return launch_rows<FmtF32, true>(a, st, parts);
}
}  // namespace sdtw
