// The slice-resident forward kernels for fp16 storage.
#include "slice_fwd.h"

namespace iabn_impl {

template bool launch_fwd_slice_dt<IABN_F16>(int, int, void*, const TileGeom&, int, const SliceArgs&,
                                            const FwdParams&, hipStream_t);

}  // namespace iabn_impl
