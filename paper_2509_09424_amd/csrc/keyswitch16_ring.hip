// The key-switch kernels of one ring, N = 4096 * 2^KS_RING: one object per ring, compiled side by side.
#include "keyswitch16_kernels.h"

template void ks16_raise<KS_RING>(ensi_ctx *, const Ks16Const &, const u64 *, size_t, int, int, u64 *, bool, hipStream_t);
template void ks16_switch<KS_RING>(ensi_ctx *, const Ks16Const &, const RotDesc *, int, u64 *, int, bool, hipStream_t, int);
