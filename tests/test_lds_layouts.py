"""The LDS that a launch is given against the layouts its tiles use.

A launch is sized for its largest leaf and its tile of most words; every tile of
any leaf in it, under any policy, workgroup width and number of actions, must
find its regions inside.  A launch that the caller captures is sized for any
policy and any number of actions.  The layouts are plain functions of a header shared by
host and device code: a small program compiled here goes through the sizes.
"""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <stdio.h>
#include "internal.hpp"
using namespace hdx;
int main() {
    long bad = 0, checked = 0;
    const int32_t odd[] = {5119, 5120, 2047, 2048, 2049, 1023, 1025};
    for (int32_t i = 0; i < 700 + 7; ++i) {
        const int32_t n = i < 700 ? 1 + i + (i > 300 ? (i - 300) * 11 : 0) : odd[i - 700];
        if (n > HDX_MAX_NAV_LEAF_SCENARIOS) continue;
        for (int32_t policy : {HDX_POLICY_DEFAULT, HDX_POLICY_RANDOM})
            for (int32_t most : {1, 3, 9}) {
                const bool stepped = policy != HDX_POLICY_DEFAULT;
                const int32_t full = nav_tile_actions(n, policy, most);
                if (n <= 1024 && full != most && bad++ < 5) printf("navigation n %d: %d actions, not %d\n", n, full, most);
                const int32_t n_max = n + (most == 3 ? 0 : 70 * most);  // of a captured launch
                for (int32_t threads = 64; threads <= 1024; threads += 64) {
                    const uint32_t given = nav_lds(n, nav_values(n, full, stepped), threads);
                    for (int32_t na = 1; na <= full; ++na) {
                        const uint32_t used = make_nav_layout((uint32_t)(na * n), (uint32_t)na, (uint32_t)(n + 63) / 64,
                                                              (uint32_t)threads / 64, stepped).total;
                        ++checked;
                        if (n_max <= HDX_MAX_NAV_LEAF_SCENARIOS && used > nav_lds(n_max, most_values(true, n_max), threads)) {
                            if (bad++ < 5) printf("navigation, captured: n %d of %d\n", n, n_max);
                        }
                        if (used > given || given > (uint32_t)kMaxDynamicLds) {
                            if (bad++ < 5) printf("navigation n %d policy %d threads %d actions %d: %u of %u\n", n, policy,
                                                  threads, na, used, given);
                        }
                    }
                }
            }
        if (n > HDX_MAX_LEAF_SCENARIOS) continue;
        for (bool two : {false, true})
            for (bool stepped : {false, true}) {
                // beside a larger leaf of either kind
                for (int32_t more : {0, 1, 63, 500}) {
                    const int32_t n_max = n + more < HDX_MAX_LEAF_SCENARIOS ? n + more : HDX_MAX_LEAF_SCENARIOS;
                    for (bool other : {false, true}) {
                        int32_t values = rock_values(n, stepped);
                        if (rock_values(n_max, other) > values) values = rock_values(n_max, other);
                        const uint32_t given = make_rock_layout(n_max, values > n_max ? values : n_max, two).total;
                        const uint32_t captured = make_rock_layout(n_max, most_values(false, n_max), two).total;
                        const uint32_t used = make_rock_layout(n, rock_values(n, stepped), two).total;
                        ++checked;
                        if (used > given || given > captured || captured > (uint32_t)kMaxDynamicLds) {
                            if (bad++ < 5) printf("rocks n %d of %d: %u of %u\n", n, n_max, used, given);
                        }
                    }
                }
            }
        if (make_ped_layout(n).total > (uint32_t)kMaxDynamicLds) ++bad;
    }
    printf("%ld checked, %ld outside\n", checked, bad);
    return bad ? 1 : 0;
}
"""


def test_every_tile_lies_inside_its_launch(tmp_path):
    src, exe = tmp_path / "layouts.cpp", tmp_path / "layouts"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_1802_06215_amd", "csrc"),
                    str(src), "-o", str(exe)], check=True)
    p = subprocess.run([str(exe)], capture_output=True, text=True)
    assert p.returncode == 0, p.stdout
    assert int(p.stdout.split()[0]) > 10000
