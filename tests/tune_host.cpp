// The launch-shape tuner (csrc/teuk_tune.hip) on the host alone: the solver, the events and the
// occupancy are stand-ins, and a step takes the time that `us_of` gives its workgroup budget.
#include <hip/hip_runtime_api.h>

#include <cmath>
#include <cstdio>
#include <functional>
#include <string>

#include "teuk_internal.h"

struct teuk_solver {
    teuk_config cfg;
    int tuned;
    bool stages;
};

static std::function<double(int)> us_of;      // < 0: the timing run fails
static bool class_fused = false;
static int default_runs = 0;
static double pending = 0, elapsed = 0;
static int failures = 0;

#define CHECK(x) (void)((x) || (++failures, std::printf("line %d: %s\n", __LINE__, #x)))

namespace teuk {
int blocked_grid(int, int) { return 512; }
int stage_grid(int, bool, int) { return 4096; }
bool steps_fused(const teuk_config& c) { return class_fused && c.workgroups == 0 && !tuned_stage_launches(c); }
}  // namespace teuk

extern "C" {
size_t teuk_footprint_bytes(const teuk_config*) { return 1; }
teuk_status teuk_create(const teuk_config* c, const teuk_device_ctx*, teuk_solver** h)
{
    *h = new teuk_solver{*c, teuk::tuned_workgroups(*c), teuk::tuned_stage_launches(*c)};
    return TEUK_OK;
}
teuk_status teuk_set_initial(teuk_solver*, const double*, int32_t) { return TEUK_OK; }
teuk_status teuk_step(teuk_solver* h, int64_t n)
{
    default_runs += h->cfg.workgroups == 0;
    if (h->cfg.workgroups == 0) CHECK(h->tuned == 0 && !h->stages);
    const double us = us_of(h->cfg.workgroups);
    pending += us * (double)n;
    return us < 0 ? TEUK_ERR_DEVICE : TEUK_OK;
}
void teuk_destroy(teuk_solver* h) { delete h; }
const char* teuk_last_error(const teuk_solver*) { return "stand-in"; }

hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { return *s = nullptr, hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { return *e = nullptr, hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return elapsed = pending, pending = 0, hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { return *ms = (float)(elapsed * 1e-3), hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "stand-in"; }
}

int main()
{
    teuk_config c{};
    c.nr = 630;
    c.ntheta = 64;
    c.integrator = TEUK_RK_SSP33;
    teuk_tune_info_t out;
    auto near = [](double a, double b) { return std::fabs(a - b) < 1e-3; };

    // A class that steps by stage launches: the time is that of the budget that is remembered, and the
    // default's that of the default budget (10 strips: 64 segments either way), however fast a run without
    // a budget might be; none is made.
    us_of = [](int wg) { return wg == 0 ? 5.0 : wg == 320 ? 9.0 : wg >= 640 ? 10.0 : 11.0; };
    CHECK(teuk_tune(&c, 7, &out) == TEUK_OK);
    CHECK(default_runs == 0);
    CHECK(out.workgroups == 320 && near(out.us_per_step, 9.0) && near(out.us_per_step_default, 10.0));
    CHECK(teuk::tuned_workgroups(c) == 320);

    // A class that steps by temporally blocked launches, faster and slower than the best budget; the run
    // without a budget does not see the shape remembered before.
    class_fused = true;
    CHECK(teuk_tune(&c, 7, &out) == TEUK_OK);
    CHECK(default_runs > 0 && near(out.us_per_step, 5.0) && near(out.us_per_step_default, 5.0));
    CHECK(!teuk::tuned_stage_launches(c));
    us_of = [](int wg) { return wg == 0 ? 12.0 : wg == 320 ? 9.0 : 10.0; };
    CHECK(teuk_tune(&c, 7, &out) == TEUK_OK);
    CHECK(near(out.us_per_step, 9.0) && near(out.us_per_step_default, 12.0));
    CHECK(teuk::tuned_stage_launches(c));

    // A run that fails leaves what was remembered.
    us_of = [](int wg) { return wg == 0 ? -1.0 : wg == 640 ? 2.0 : 3.0; };
    CHECK(teuk_tune(&c, 7, &out) == TEUK_ERR_DEVICE);
    CHECK(teuk::tuned_workgroups(c) == 320 && teuk::tuned_stage_launches(c));
    std::printf("failures %d\n", failures);
    return failures != 0;
}
