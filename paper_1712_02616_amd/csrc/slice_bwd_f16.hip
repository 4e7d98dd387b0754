// The slice-resident backward kernels for fp16 storage.
#include "slice_bwd.h"

namespace iabn_impl {

template bool launch_bwd_slice_dt<IABN_F16>(int, int, bool, const void*, const void*, void*,
                                            const TileGeom&, int, const SliceArgs&, const BwdParams&,
                                            hipStream_t);

}  // namespace iabn_impl
