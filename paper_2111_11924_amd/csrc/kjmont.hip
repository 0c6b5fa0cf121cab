// Blinded decryption in one pass per prime with Montgomery products, one lane per
// number (halves_joint_unit), of the 1024- to 4096-bit classes: as kmont.inc for
// the plain halves.  Products align each column (mont.hpp), as in kjoint.hip.
#define PMK_COLUMN_ALIGN 1
#include <algorithm>

#include "kernels_impl.hpp"

namespace pmk {

template <int CB>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2))) void halves_joint_mont_kernel(
    ClassRun r, uint64_t slot_words, uint32_t u_begin, uint32_t u_end) {
    code_align<code_id(kCodeJointMont, CB, 0)>();
    uint32_t *tbl = r.table + (size_t)blockIdx.x * slot_words;
    __shared__ uint32_t lds[lds_words_dec<CB>()];
    for (uint32_t u = u_begin + blockIdx.x; u < u_end; u += gridDim.x) halves_joint_unit<CB>(r, u, tbl, lds);
}

namespace {

template <int CB>
uint32_t resident() {
    static const uint32_t nb = [] {
        int n = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, (const void *)halves_joint_mont_kernel<CB>, 64, 0) !=
                hipSuccess ||
            n < 1)
            n = 1;
        return (uint32_t)n;
    }();
    return nb * (uint32_t)device_cus();
}

template <int CB>
int launch(const ClassRun &r, hipStream_t s) {
    const uint64_t slot = 2 * table_words_per_slot(r.cls, 1, r.win);  // two odd-power tables
    return launch_rounds(r, slot, resident<CB>(), [&](uint32_t blocks, uint32_t from, uint32_t to) {
        hipLaunchKernelGGL(halves_joint_mont_kernel<CB>, dim3(blocks), dim3(64), 0, s, r, slot, from, to);
        return (int)hipGetLastError();
    });
}

}  // namespace

uint32_t joint_mont_resident(int cls) {
    switch (kClassBits[cls]) {
        case 1024: return resident<1024>();
        case 2048: return resident<2048>();
        case 3072: return resident<3072>();
        case 4096: return resident<4096>();
        default: return 0;
    }
}

int launch_joint_mont(const ClassRun &r, void *stream) {
    hipStream_t s = (hipStream_t)stream;
    switch (kClassBits[r.cls]) {
        case 1024: return launch<1024>(r, s);
        case 2048: return launch<2048>(r, s);
        case 3072: return launch<3072>(r, s);
        case 4096: return launch<4096>(r, s);
        default: return (int)hipErrorInvalidValue;
    }
}

}  // namespace pmk
