// The column form of the temporal sweep for compensated 16-bit storage.
#include "column.h"

namespace fdtd {

template hipError_t launch_column_step<f16c>(const Geom &, const Fields<f16c> &, const Fields<f16c> &,
                                                const Coefs<float> &, int, int, hipStream_t, unsigned *);
template hipError_t launch_column_step<bf16c>(const Geom &, const Fields<bf16c> &, const Fields<bf16c> &,
                                                const Coefs<float> &, int, int, hipStream_t, unsigned *);

}  // namespace fdtd
