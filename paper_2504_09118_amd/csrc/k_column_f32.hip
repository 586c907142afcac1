// The column form of the temporal sweep for FP32 storage.
#include "column.h"

namespace fdtd {

template hipError_t launch_column_step<float>(const Geom &, const Fields<float> &, const Fields<float> &,
                                                const Coefs<float> &, int, int, hipStream_t, unsigned *);

}  // namespace fdtd
