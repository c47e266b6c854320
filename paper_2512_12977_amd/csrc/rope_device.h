// Device arithmetic shared by the kernels that rotate queries and keys.
#ifndef VLC_ROPE_DEVICE_H_
#define VLC_ROPE_DEVICE_H_

#include <hip/hip_runtime.h>

namespace vlc {

// sin/cos of delta * inv_freq.  The angle is formed and reduced to [-pi, pi] in double (positions
// reach tens of thousands of radians, beyond what a float angle resolves), then evaluated in float.
// FAST (bf16 storage, 8 significant bits): the hardware sine/cosine, which take the angle in
// revolutions; otherwise the library routines on the reduced angle.
template <bool FAST>
__device__ __forceinline__ void rope_sincos(double inv_freq, int delta, float* s, float* c) {
  double rev = (double)delta * inv_freq * 0.15915494309189535;   // angle / 2pi
  rev -= rint(rev);
  if (FAST) {
    *s = __builtin_amdgcn_sinf((float)rev);
    *c = __builtin_amdgcn_cosf((float)rev);
  } else {
    const float r = (float)(rev * 6.283185307179586);
    *s = sinf(r);
    *c = cosf(r);
  }
}

}  // namespace vlc
#endif
