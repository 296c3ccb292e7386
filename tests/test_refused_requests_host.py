"""Host requests that are refused by a frame's own counts: none of the frame's
windows may be read first, since its window count is as untrustworthy as the
rest.  The windows lie at the end of a readable page and the next page is
unreadable, so a walk over n_windows of them ends the program."""
import subprocess

from tests.hostbuild import host_program

PROGRAM = r"""
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdio.h>
#include <string.h>
#include <sys/mman.h>
#include "runtime.h"
using namespace dpps;

int main()
{
    char *mem = (char *)mmap(nullptr, 8192, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
    if (mem == (char *)MAP_FAILED || mprotect(mem + 4096, 4096, PROT_NONE)) return 2;
    dpps_window *win = (dpps_window *)(mem + 4096) - 1;
    *win = {0.2f, 0, 0, 61, 46};
    dpps_robot robots[4] = {};
    dpps_variant variants[2] = {{DPPS_FLAT, 3.0f}, {DPPS_FLAT, 4.0f}};
    dpps_ctx c;
    memset(&c.p, 0, sizeof c.p);
    c.p.field_len = 12.0f;
    c.p.field_wid = 9.0f;
    dpps_frame good;
    memset(&good, 0, sizeof good);
    good.n_team = good.n_opp = 2;
    good.n_variants = 2;
    good.n_windows = 0x7FFFFFFF;
    OneFrame one;
    for (int k = 0; k < 12; ++k) {
        dpps_frame f = good;
        const dpps_robot *r = robots;
        const dpps_variant *v = variants;
        int want = DPPS_E_INVALID;
        switch (k) {
        case 0: f.n_team = 0; break;
        case 1: f.n_team = DPPS_MAX_SIDE + 1; break;
        case 2: f.n_opp = -1; break;
        case 3: f.passer = 2; break;
        case 4: f.n_variants = 0; break;
        case 5: f.n_variants = DPPS_MAX_VARIANTS + 1; want = DPPS_E_UNSUPPORTED; break;
        case 6: f.robot_off = -1; break;
        case 7: f.variant_off = -1; break;
        case 8: f.ball_x = NAN; break;
        case 9: f.out_off = -1; break;
        case 10: r = nullptr; break;
        case 11: v = nullptr; break;
        }
        const int rc = stage_batch(&c, &c.scratch, 1, &f, r, win, v, one, nullptr);
        printf("case %d: %d, expected %d\n", k, rc, want);
        fflush(stdout);
        if (rc != want) return 1;
    }
    return 0;
}
"""


def test_bad_counts_are_refused_before_the_windows_are_read(tmp_path):
    exe = host_program(tmp_path, PROGRAM)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, (r.returncode, r.stdout, r.stderr)
    assert r.stdout.count("case") == 12
