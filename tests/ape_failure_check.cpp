// The host side of smear.hip against stand-ins for the device: allocations and
// launches that fail when they are told to (tests/test_ape_failure.py).  A call to
// qcd_field_ape_smear that fails must leave the handle as it was.
#include <cstdio>

#include "smear.hip"

namespace {
bool scratch_fails, links_fail, launch_fails;
char memory[2];   // addresses of the scratch and of the links
int allocated, freed, errors;
void expect(bool ok, const char *what) {
    if (!ok) {
        std::fprintf(stderr, "mismatch: %s\n", what);
        ++errors;
    }
}
}  // namespace

namespace dfl {
int set_error(int code, const std::string &) { return code; }
int field_buffer(qcd_field, int, size_t, void **p) {
    *p = memory;
    return scratch_fails ? (int)QCD_ENOMEM : 0;
}
bool dev_alloc(int, void **p, size_t) {
    if (links_fail) return false;
    ++allocated;
    *p = memory + 1;
    return true;
}
ProfScope::ProfScope(int, hipStream_t, double, double, double) {}
ProfScope::~ProfScope() {}
}  // namespace dfl

extern "C" {
hipError_t hipFree(void *p) {
    if (p) ++freed;
    return hipSuccess;
}
hipError_t hipGetLastError(void) { return launch_fails ? hipErrorLaunchFailure : hipSuccess; }
const char *hipGetErrorString(hipError_t) { return ""; }
hipError_t hipLaunchKernel(const void *, dim3, dim3, void **, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3 *, dim3 *, size_t *, hipStream_t *) { return hipSuccess; }
void **__hipRegisterFatBinary(const void *) { return nullptr; }
void __hipRegisterFunction(void **, const void *, char *, const char *, unsigned, void *, void *, void *, void *, int *) {}
void __hipUnregisterFatBinary(void **) {}
}

int main() {
    for (int iters = 0; iters < 4; ++iters)
        for (int what = 0; what < 4; ++what) {
            qcd_field_s f{};
            f.g.L[0] = f.g.L[1] = f.g.L[2] = f.g.L[3] = 4;
            f.g.V = 256;
            allocated = freed = 0;
            scratch_fails = what == 1;
            links_fail = what == 2;
            launch_fails = what == 3;
            const int rc = qcd_field_ape_smear(&f, 0.5, iters, nullptr);
            // without steps there is no scratch to fail
            const bool fails = what == 2 || what == 3 || (what == 1 && iters > 0);
            expect((rc < 0) == fails, "status of a first call");
            expect((f.Uape == nullptr) == fails, "links of a handle that had none");
            expect(allocated - freed == (fails ? 0 : 1), "links freed by a first call that fails");
            launch_fails = false;
            char out;
            expect(qcd_field_get_ape_links(&f, &out, nullptr) == (fails ? (int)QCD_ENOTSET : 0), "use after it");
            expect(gauss_smear(&f, &out, &out, 1, QCD_F64, 0.1, 0, nullptr) ==
                       (fails ? (int)QCD_ENOTSET : scratch_fails ? (int)QCD_ENOMEM : 0), "smearing after it");

            // a handle that has links keeps them
            char kept;
            f.Uape = &kept;
            allocated = freed = 0;
            launch_fails = what == 3;
            const int again = qcd_field_ape_smear(&f, 0.5, iters, nullptr);
            expect((again < 0) == (what == 3 || (what == 1 && iters > 0)), "status of a second call");
            expect(f.Uape == &kept && allocated == 0 && freed == 0, "links of a handle that had some");
        }
    return errors ? 1 : 0;
}
