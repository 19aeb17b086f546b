// A CPU build of the library's host side (api.cpp, plan.cpp, lse_merge.hip) in
// which every launch is recorded and none is made, on a device of 256 compute
// units.
#include <hip/hip_runtime.h>

#include <vector>

#include "internal.h"

namespace {
std::vector<mocap::AttnLaunch> attn;  // of the attention launches, in order
std::vector<unsigned> dims;           // grid and block of the merge launches, 6 numbers each
int launches = 0;
}  // namespace

namespace mocap {
hipError_t launch_chunk_attn(const AttnLaunch& p, int, hipStream_t) {
  ++launches;
  attn.push_back(p);
  return hipSuccess;
}
hipError_t launch_chunk_attn_short(const AttnLaunch& p, int d, hipStream_t s) { return launch_chunk_attn(p, d, s); }
hipError_t launch_kv_append(const AppendLaunch&, int, hipStream_t) {
  ++launches;
  return hipSuccess;
}
}  // namespace mocap

extern "C" {

hipError_t hipGetDevice(int* dev) {
  *dev = 0;
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* value, hipDeviceAttribute_t, int) {
  *value = 256;
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** ptr, const void*) {
  *ptr = (void*)0x100000;
  return hipSuccess;
}
// A kernel<<<grid, block>>> call passes its configuration here first.
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t, hipStream_t) {
  ++launches;
  for (unsigned x : {grid.x, grid.y, grid.z, block.x, block.y, block.z}) dims.push_back(x);
  return hipErrorUnknown;  // not 0: the launch itself is left out
}
hipError_t hipGetLastError() { return hipSuccess; }

int record_launches() { return launches; }
// The last attention launch: placement, ranges, workgroups.
void record_last(int* out) {
  out[0] = attn.back().pairing;
  out[1] = attn.back().n_ranges;
  out[2] = attn.back().total_wgs;
}
// The last merge launch: grid and block.
void record_merge(unsigned* out) {
  for (int i = 0; i < 6; ++i) out[i] = dims[dims.size() - 6 + i];
}

}  // extern "C"
