// What the entry points of the library launch, without a GPU: lba_kernels.hip and lba_plan.cpp as they are, and in place of every
// kernel launcher one that keeps the plan it is given.  tests/test_launched_plans_cpu.py builds and loads it.
#include "lba_launch.h"

namespace {
lba::Plan last;
const char* launcher = "";
hipError_t keep(const lba::Plan& pl, const char* name) {
    last = pl;
    launcher = name;
    return hipSuccess;
}
}  // namespace

namespace lba {
#define LBA_KEEP(NAME) hipError_t NAME(const Plan& pl, hipStream_t) { return keep(pl, #NAME); }
LBA_KEEP(launch_fast_44) LBA_KEEP(launch_fast_24) LBA_KEEP(launch_fast_22) LBA_KEEP(launch_fast_amode) LBA_KEEP(launch_fast_mixed)
LBA_KEEP(launch_fast_conv) LBA_KEEP(launch_fast_in_mixed_seq) LBA_KEEP(launch_fast_in_mixed_chunk) LBA_KEEP(launch_fast_odd) LBA_KEEP(launch_kpar)
LBA_KEEP(launch_fast_bwd) LBA_KEEP(launch_half) LBA_KEEP(launch_half_conv) LBA_KEEP(launch_wide) LBA_KEEP(launch_wide_conv)
LBA_KEEP(launch_fast_staged) LBA_KEEP(launch_half_bwd) LBA_KEEP(launch_half_alone) LBA_KEEP(launch_half_bwd_alone) LBA_KEEP(launch_fast_diff)
LBA_KEEP(launch_gen)
int brick_maps_fill(void*, int64_t, int64_t, int64_t, bool, hipStream_t) { return LBA_OK; }
int brick_maps_scan(const uint32_t*, void*, int64_t, int64_t, int64_t, uint32_t, hipStream_t) { return LBA_OK; }
void brick_map_params(void*, int64_t, int64_t, int64_t, KParams*) {}
}  // namespace lba

extern "C" {
size_t lba_grad_workspace_bytes(int64_t, int64_t, int64_t) { return 256; }
struct launched { int32_t grid_x, grid_y, tm, tn, mix_main, mix_half, mix_tail, mix_tail16, packed, staged, alone, of_only, kpar; };
// the launcher of the last call that launched, and its plan; the record is empty again afterwards
const char* take_launched(launched* out) {
    const lba::KParams& kp = last.kp;
    *out = {last.grid_x, last.grid_y, last.tm, last.tn, kp.mix_main, kp.mix_half, last.mix_tail, kp.mix_tail16, kp.h_on, last.staged, last.alone, last.of_only, last.kpar};
    const char* const name = launcher;
    launcher = "";
    return name;
}
}  // extern "C"
