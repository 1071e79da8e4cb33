// What fake_hip.c has to know of the device properties.
#define __HIP_PLATFORM_AMD__
#include <hip/hip_runtime_api.h>

#include <cstddef>
extern "C" {
extern const size_t fake_arch_offset = offsetof(hipDeviceProp_t, gcnArchName), fake_prop_bytes = sizeof(hipDeviceProp_t);
}
