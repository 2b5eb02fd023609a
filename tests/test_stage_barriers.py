"""The INT8 projection kernels load the next chunk into an LDS stage right after a barrier, while the
waves' last reads of that stage came before it. The barrier orders these only if every wave has waited
for its own LDS reads (and for its loads into the other stage) first: without that wait in the source,
the scheduler may move it past the barrier. Read off the gfx950 code that the build made."""
import os
import re
import subprocess

import pytest

from paper_2609_29499_amd import build as BLD

LLVM = "/opt/rocm/llvm/bin"


def _kernels(tmp_path):
    """{kernel name: its instructions} of the built prefill_i8 object."""
    obj = os.path.join(BLD.OBJ, "prefill_i8.o")
    if not (os.path.exists(obj) and os.path.exists(f"{LLVM}/llvm-objdump")):
        pytest.skip("no built object or no llvm-objdump")
    link = tmp_path / "prefill_i8.o"
    os.symlink(obj, link)
    subprocess.run([f"{LLVM}/llvm-objdump", "--offloading", str(link)], check=True, capture_output=True, cwd=tmp_path)
    dev = [f for f in os.listdir(tmp_path) if "gfx950" in f]
    assert len(dev) == 1
    text = subprocess.run([f"{LLVM}/llvm-objdump", "-d", "--mcpu=gfx950", str(tmp_path / dev[0])], check=True,
                          capture_output=True, text=True).stdout
    out, name = {}, None
    for line in text.splitlines():
        m = re.match(r"^[0-9a-f]+ <(.*)>:", line)
        if m:
            name = m.group(1)
            out[name] = []
        elif name and line.strip():
            out[name].append(line.split("//")[0].strip())
    return {n: i for n, i in out.items() if "pf_i8_kernel" in n}


def test_stage_barriers_follow_a_wait_for_lds_reads(tmp_path):
    kernels = _kernels(tmp_path)
    assert len(kernels) == 30          # three modes, five tile shapes, two stores
    for name, ins in kernels.items():
        at = [i for i, t in enumerate(ins) if t.startswith("s_barrier")] + [len(ins)]
        # the barriers behind which loads into LDS are issued
        stage = [i for i, end in zip(at, at[1:])
                 if any(t.startswith("buffer_load") and t.endswith(" lds") for t in ins[i:end])]
        assert len(stage) >= 2 or "Li1ELi1ELi4E" in name, name     # (one wave's group shares its stages with no other)
        for i in stage:
            # between the barrier and the wait before it: no LDS access, and the wait covers LDS
            j = next(j for j in range(i - 1, -1, -1) if ins[j].startswith("s_waitcnt"))
            assert "lgkmcnt(0)" in ins[j], f"{name}: {ins[j]} before a barrier"
            assert not any(t.startswith("ds_") for t in ins[j:i]), name
