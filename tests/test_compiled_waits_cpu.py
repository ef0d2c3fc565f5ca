"""Waits that the prompt kernels need and the compiler does not see to, looked for in the assembly they compile to."""
import concurrent.futures
import os
import re
import shutil
import subprocess

import pytest

from paper_2406_12335_amd import build

SOURCES = ["prefill_wide.hip", "prefill_mfma.hip", "prefill_direct.hip"]


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{kernel: its instructions in order}; a label is an instruction ending in a colon."""
    if not (shutil.which("hipcc") or os.path.exists("/opt/rocm/bin/hipcc")):
        pytest.skip("hipcc not found")
    out = tmp_path_factory.mktemp("asm")

    def compile_one(name):
        asm = str(out / (name + ".s"))
        subprocess.check_call([build.hipcc(), *build.HIPCC_FLAGS, *build.EXTRA_FLAGS.get(name, []), "--cuda-device-only", "-S",
                               os.path.join(build.CSRC, name), "-o", asm], stderr=subprocess.DEVNULL)
        with open(asm) as f:
            return f.read()

    with concurrent.futures.ThreadPoolExecutor(len(SOURCES)) as pool:
        texts = list(pool.map(compile_one, SOURCES))
    found, body = {}, None
    for line in "\n".join(texts).splitlines():
        text = line.split(";")[0].strip()
        if re.match(r"_ZN\S+:$", text):
            body = found.setdefault(text[:-1], [])
        elif text.startswith(".Lfunc_end"):
            body = None
        elif body is not None and re.match(r"(v|s|ds|global|buffer|flat|scratch)_|\.LBB\S+:$", text):
            body.append(text)
    assert len(found) > 20
    return found


def test_lds_reads_are_complete_before_a_barrier(kernels):
    """Behind a barrier other wavefronts write what was read before it."""
    for name, body in kernels.items():
        for i, text in enumerate(body):
            if text != "s_barrier":
                continue
            before = next(x for x in reversed(body[:i]) if x.startswith(("ds_", "s_waitcnt")) and ("lgkmcnt" in x or x.startswith("ds_")))
            assert "lgkmcnt(0)" in before, "%s: %s reaches the barrier at instruction %d" % (name, before, i)
