"""The team barrier of the one-launch refinement, as compiled for gfx950: every
wave waits for its own stores before the workgroup barrier behind which one
thread counts the workgroup in.

A workgroup barrier alone does not wait for stores, and the counting thread's
own wait covers its own wave only, so without the wait another workgroup could
pass the team barrier and read a value whose store is still on its way.  The
check reads the assembly of a two-line kernel around the barrier, built here.
"""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

SOURCE = """
#include "team.h"
using namespace kktlu;
__global__ void k_probe(unsigned int* t, int* stall, double* a, double* b, double* c) {
  FgTeam tm{t, blockIdx.x, gridDim.x, 0u, stall};
  a[blockIdx.x * blockDim.x + threadIdx.x] = 1.0;
  if (!fg_team_sync(tm, [&] { b[threadIdx.x] = 2.0; })) return;
  c[threadIdx.x] = a[threadIdx.x] + b[threadIdx.x];
}
"""


# the barrier without a reduction, and the one in front of plain loads
PLAIN = SOURCE.replace("fg_team_sync(tm, [&] { b[threadIdx.x] = 2.0; })", "fg_team_sync(tm)")
ACQUIRE = SOURCE.replace("fg_team_sync(tm, [&] { b[threadIdx.x] = 2.0; })",
                         "fg_team_sync<true>(tm)")


def assembly(tmp_path, source):
    src = tmp_path / "probe.hip"
    src.write_text(source)
    out = tmp_path / "probe.s"
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "--offload-device-only",
                    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-S",
                    "-I", os.path.join(ROOT, "paper_2306_14337_amd", "csrc"), str(src),
                    "-o", str(out)], check=True, capture_output=True, text=True)
    body = out.read_text().split("k_probe", 1)[1].split("s_endpgm")
    return [ln.strip() for part in body for ln in part.splitlines()]


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="no hipcc")
def test_every_wave_waits_for_its_stores(tmp_path):
    lines = assembly(tmp_path, SOURCE)
    # vector stores of doubles: the kernel's own (a before the barrier, b in
    # fin, c behind it); counters and flags are single words
    stores = [i for i, ln in enumerate(lines)
              if re.match(r"global_store_dwordx2|flat_store_dwordx2", ln)]
    assert len(stores) == 3
    for i in sorted(stores)[:2]:
        barrier = next(k for k in range(i, len(lines)) if lines[k].startswith("s_barrier"))
        between = lines[i + 1:barrier]
        assert any(re.search(r"s_waitcnt.*vmcnt\(0\)", ln) for ln in between), between


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="no hipcc")
@pytest.mark.parametrize("source,invalidates", [(PLAIN, False), (ACQUIRE, True)])
def test_no_cache_is_written_back_without_a_reduction(tmp_path, source, invalidates):
    """What passes from phase to phase is device-coherent: a barrier moves no
    cache contents, but for the invalidation in front of plain loads."""
    lines = assembly(tmp_path, source)
    assert not any(ln.startswith("buffer_wbl2") for ln in lines)
    assert any(ln.startswith("buffer_inv") for ln in lines) == invalidates
    store = next(i for i, ln in enumerate(lines) if re.match(r"global_store_dwordx2", ln))
    barrier = next(k for k in range(store, len(lines)) if lines[k].startswith("s_barrier"))
    assert any(re.search(r"s_waitcnt.*vmcnt\(0\)", ln) for ln in lines[store:barrier])


def test_a_team_outwaits_a_batch_refactorization():
    """Launches of other streams hold the chip for some milliseconds; a team
    closed within them would be a few workgroups.  A poll takes about 1 us."""
    text = open(os.path.join(ROOT, "paper_2306_14337_amd", "csrc", "team.h")).read()
    assert int(re.search(r"FG_TEAM_POLLS = (\d+);", text).group(1)) >= 5000
