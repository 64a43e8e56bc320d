"""lora_thin_kernel waits for its own direct-to-LDS loads by counting the loads issued after them, which holds only for the order that
the source states.  Checked in the code that the compiler makes of it, for every instantiation: 2 RB loads of X per chunk and wave, 2 NB
of the factors."""
import os
import re
import subprocess

import pytest

from paper_2510_06710_amd import build


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{(RB, NB): its loads, waits, barriers and matrix instructions in order}."""
    out = tmp_path_factory.mktemp("asm") / "lora_grad.s"
    subprocess.run([build.HIPCC, *build.FLAGS, "-S", "--cuda-device-only", os.path.join(build.CSRC, "lora_grad.hip"), "-o", str(out)],
                   check=True, capture_output=True)
    found = {}
    for m in re.finditer(r"^_ZN\S*lora_thin_kernelILi(\d)ELi(\d)E[^\n]*:[^\n]*\n(.*?)^\s*s_endpgm", out.read_text(), re.M | re.S):
        lines = [x.strip() for x in m.group(3).splitlines()]
        found[int(m.group(1)), int(m.group(2))] = [x for x in lines if re.match(r"(buffer_load|global_load|s_waitcnt|s_barrier|v_mfma)", x)]
    return found


def test_the_first_chunk_is_loaded_first(kernels):
    """The wait for chunk 0 leaves as many loads in flight as chunk 1 and the first factors are."""
    assert sorted(kernels) == [(rb, nb) for rb in (1, 2) for nb in range(1, 9)]
    for (rb, nb), ops in kernels.items():
        before = [x for x in ops[:ops.index("s_barrier")] if "_load" in x]
        assert len(before) == 4 * rb + 2 * nb and all(x.endswith(" lds") for x in before[: 2 * rb]), (rb, nb, before)
        assert sum(x.endswith(" lds") for x in before) == 4 * rb, (rb, nb, before)


def test_no_step_waits_for_the_loads_behind_its_own(kernels):
    """In the loop every wait leaves the next chunk's loads and factors in flight: the ring is three chunks deep."""
    for (rb, nb), ops in kernels.items():
        last = max(i for i, x in enumerate(ops) if x.startswith("v_mfma"))
        waits = [int(n) for x in ops[ops.index("s_barrier"):last] for n in re.findall(r"vmcnt\((\d+)\)", x)]
        assert waits and min(waits) >= 2 * rb + 2 * nb, (rb, nb, waits)
