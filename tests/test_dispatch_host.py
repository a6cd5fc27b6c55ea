"""The launch dispatch (csrc/fdetd_dispatch.cpp) on the host, with the kernels' entry points replaced by recorders: a
group of envelope stages reaches the FP64 launch of its width with its own arguments, widths without a group kernel are
refused, and so are a stage's arguments that carry the group's role (they end before a group's fields)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2605_12132_amd", "csrc")

PROGRAM = r'''
#include "fdetd_envelope.h"
#include <cstdio>
#include <cstring>
namespace fdetd {
int width, precision, role, seg;
#define STUB_ND(N)                                                                                        \
    template <> hipError_t march_maxwell_nd<N>(int, const BatchArgs &, hipStream_t) { return hipErrorInvalidValue; } \
    template <> hipError_t march_stagger_nd<N>(int, const BatchArgs &, hipStream_t) { return hipErrorInvalidValue; } \
    template <> hipError_t march_envelope_nd<N>(int prec, const BatchArgs &a, hipStream_t)               \
    {                                                                                                    \
        width = N; precision = prec; role = a.role;                                                      \
        if (a.role == ROLE_ENV_GROUP) seg = static_cast<const EnvFuseArgs &>(a).seg;                     \
        return hipSuccess;                                                                               \
    }
STUB_ND(1) STUB_ND(2) STUB_ND(3) STUB_ND(4) STUB_ND(5) STUB_ND(6) STUB_ND(7) STUB_ND(8)
STUB_ND(9) STUB_ND(10) STUB_ND(11) STUB_ND(12) STUB_ND(13) STUB_ND(14) STUB_ND(15) STUB_ND(16)
hipError_t march_maxwell_any_p64(const BatchArgs &, hipStream_t) { return hipErrorInvalidValue; }
hipError_t march_maxwell_any_p32(const BatchArgs &, hipStream_t) { return hipErrorInvalidValue; }
hipError_t march_maxwell_any_p32c(const BatchArgs &, hipStream_t) { return hipErrorInvalidValue; }
hipError_t march_stagger_any_p64(const BatchArgs &, hipStream_t) { return hipErrorInvalidValue; }
hipError_t march_stagger_any_p32(const BatchArgs &, hipStream_t) { return hipErrorInvalidValue; }
}
using namespace fdetd;
int main() {
    EnvFuseArgs g{};
    g.seg = 77;
    for (int nd = 1; nd <= 16; ++nd) {
        width = seg = 0;
        const hipError_t e = launch_envelope_group(nd, g, nullptr);
        if (nd <= kEnvFuseND ? e != hipSuccess || width != nd || precision != P64 || role != ROLE_ENV_GROUP || seg != 77
                             : e == hipSuccess || width) return printf("FAIL group %d\n", nd), 1;
        for (int prec : {P64, P32}) {
            BatchArgs *a = new BatchArgs();  // an allocation of its own: the sanitizer sees a read past it
            width = 0;
            if (launch_envelope_march(prec, nd, *a, nullptr) != hipSuccess || width != nd || precision != prec)
                return printf("FAIL stage %d\n", nd), 1;
            a->role = ROLE_ENV_GROUP;
            width = 0;
            if (launch_envelope_march(prec, nd, *a, nullptr) == hipSuccess || width) return printf("FAIL role %d\n", nd), 1;
            delete a;
        }
    }
    printf("dispatch ok\n");
}
'''


def test_groups_have_their_own_launch(tmp_path):
    src, exe = tmp_path / "t.cpp", str(tmp_path / "t")
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-fsanitize=address,undefined", "-D__HIP_PLATFORM_AMD__", "-I",
                    "/opt/rocm/include", "-I", os.path.join(ROOT, "include"), "-I", CSRC, str(src),
                    os.path.join(CSRC, "fdetd_dispatch.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "dispatch ok" in r.stdout, r.stdout + r.stderr
