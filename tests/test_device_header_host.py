"""Host checks of the device-side headers: facts that hold at compile time,
asked of the compiler (nothing runs on a GPU)."""
import subprocess
from pathlib import Path

from paper_2411_06405_amd import build as B

CSRC = Path(B.__file__).resolve().parent / "csrc"


def _compile(src, tmp_path, arch="gfx950", device=False):
    f = tmp_path / "probe.hip"
    f.write_text(src)
    side = "--cuda-device-only" if device else "--cuda-host-only"
    return subprocess.run([B.HIPCC, "-std=c++17", f"--offload-arch={arch}", side, "-fsyntax-only",
                           "-I", str(CSRC), str(f)], capture_output=True, text=True)


def test_a_team_never_outgrows_its_arrays(tmp_path):
    r = _compile("""
#include "hotruss_dev.h"
using namespace hotruss;
constexpr uint32_t FLAGS = sizeof(Team::flag) / 4, MINS = sizeof(Team::smin) / 4, COUNTS = sizeof(Team::scnt) / 4;
static_assert(FLAGS == TEAM_MAX && MINS == TEAM_MAX && COUNTS == TEAM_MAX, "");
static_assert(TEAM_MAX <= WAVE, "one lane a member");
static_assert(team_admits(1) && team_admits(TEAM_MAX - 1), "");
static_assert(!team_admits(TEAM_MAX) && !team_admits(TEAM_CLOSED) && !team_admits(TEAM_CLOSED + 300), "");
static_assert(team_size(1) == 1 && team_size(TEAM_MAX) == TEAM_MAX && team_size(TEAM_MAX + 1) == TEAM_MAX, "");
static_assert(team_size(TEAM_CLOSED - 1) == TEAM_MAX, "");
""", tmp_path)
    assert r.returncode == 0, r.stderr[-2000:]


def test_device_code_is_tied_to_its_chip(tmp_path):
    src = '#include "hotruss_dev.h"\n'
    assert _compile(src, tmp_path, device=True).returncode == 0
    r = _compile(src, tmp_path, arch="gfx942", device=True)
    assert r.returncode != 0 and "gfx950" in r.stderr
