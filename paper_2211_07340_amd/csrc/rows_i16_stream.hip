// The row-lane kernel on int16 references, extending resident rows (see rows.h).
#include "rows.h"

namespace sdtw {
hipError_t launch_rows_i16_stream(const RowsArgs& a, hipStream_t st, int parts) {
  return launch_rows<FmtI16, true>(a, st, parts);
}
}  // namespace sdtw
