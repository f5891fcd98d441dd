"""Words that tell another workgroup that something is in memory: in the
generated code, the wave waits for its stores and atomics (vmcnt(0)) before it
writes them.  Read from the assembly of the kernels, since no run on the GPU
shows a missing wait reliably."""
import os
import re
import subprocess

import pytest

from paper_2212_07597_amd import _build

pytestmark = pytest.mark.skipif(not os.path.exists(_build.HIPCC), reason="no hipcc")

WAIT = re.compile(r"s_waitcnt.*vmcnt\(0\)")
WRITE = re.compile(r"(global|flat|buffer|scratch)_(store|atomic)")


def kernel(tmp_path_factory, source, name):
    """Instructions of the kernel whose mangled name holds ``name``."""
    out = tmp_path_factory.mktemp("asm") / "k.s"
    flags = [f for f in _build.HIP_FLAGS if f not in ("-shared", "-fPIC")]
    subprocess.run([_build.HIPCC, *flags, "-I", os.path.join(_build.ROOT, "include"), "--cuda-device-only", "-S", "-o",
                    str(out), os.path.join(_build.PKG, "csrc", source)], check=True, capture_output=True)
    body, inside = [], False
    for line in out.read_text().split("\n"):
        label = re.match(r"(_Z\w+):", line)
        if label:
            inside = name in label.group(1)
        elif inside and re.match(r"\s+[a-z]\w+", line):
            body.append(line.strip())
    assert body, name
    return body


def only(body, pattern):
    at = [i for i, x in enumerate(body) if re.match(pattern, x)]
    assert len(at) == 1, (pattern, [body[i] for i in at])
    return at[0]


def waited(body, at):
    """Nothing is written between the last wait for stores and ``at``."""
    for x in reversed(body[:at]):
        if WAIT.match(x):
            return True
        if WRITE.match(x):
            return False
    return False


@pytest.mark.parametrize("waves", [8, 16])
def test_rate_finish(tmp_path_factory, waves):
    """Every wave's counts and flags before the barrier in front of the count
    of finished workgroups (header word 1)."""
    body = kernel(tmp_path_factory, "rate.hip", f"k_rateILi{waves}E")
    done = only(body, r"global_atomic_add_x2 .*offset:8 sc0")
    barrier = max(i for i in range(done) if body[i].startswith("s_barrier"))
    assert waited(body, barrier)


def test_tile_map_chain(tmp_path_factory):
    """A tile's map before its mark, the mark before the chain is asked for, the
    chain's exits and position before it is free, and free before the marks are
    read again."""
    body = kernel(tmp_path_factory, "sampler_kernels.hip", "6k_tmap")
    ask = only(body, r"global_atomic_swap_x2 .* sc0")
    assert waited(body, ask)
    mark = max(i for i in range(ask) if WRITE.match(body[i]))
    assert body[mark].startswith("global_store_dwordx2") and body[mark].endswith("sc1")
    assert waited(body, mark)
    position = only(body, r"global_store_dword .* sc1")  # (the only 32-bit word stored through to memory)
    free = min(i for i in range(position + 1, len(body)) if WRITE.match(body[i]))
    assert body[free].startswith("global_store_dwordx2") and body[free].endswith("sc1")
    assert waited(body, free)
    look = min(i for i in range(free + 1, len(body)) if body[i].startswith("global_load"))
    assert any(WAIT.match(x) for x in body[free + 1:look])
