// The column form of the temporal sweep for FP16 and BF16 storage.
#include "column.h"

namespace fdtd {

template hipError_t launch_column_step<f16>(const Geom &, const Fields<f16> &, const Fields<f16> &,
                                                const Coefs<float> &, int, int, hipStream_t, unsigned *);
template hipError_t launch_column_step<bf16>(const Geom &, const Fields<bf16> &, const Fields<bf16> &,
                                                const Coefs<float> &, int, int, hipStream_t, unsigned *);

}  // namespace fdtd
