"""Waits that the kernels need and the compiler does not always see to, looked for in the assembly they compile to."""
import concurrent.futures
import os
import re
import shutil
import subprocess

import pytest

from paper_2406_12335_amd import build

SOURCES = ["prefill_onepass.hip", "prefill_wide.hip", "prefill_mfma.hip", "prefill_direct.hip", "decode.hip"]


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


# Wait states (instructions, s_nop n for n + 1) between an MFMA and a vector or memory instruction that reads its result: the passes it
# takes and 3, on gfx950 one more, for bf16 inputs; the passes and 2 for float ones.
WAIT_STATES = {"v_mfma_f32_32x32x16_bf16": 12, "v_mfma_f32_16x16x32_bf16": 8, "v_mfma_f32_32x32x2_f32": 18, "v_mfma_f32_32x32x2f32": 18}


def _registers(operand):
    m = re.match(r"-?\|?v(?:\[(\d+):(\d+)\]|(\d+)\b)", operand.strip())
    if not m:
        return set()
    return {int(m.group(3))} if m.group(3) else set(range(int(m.group(1)), int(m.group(2)) + 1))


def _read_by(text):
    op, _, rest = text.partition(" ")
    operands = rest.split(",")
    if "mfma" in op:                                       # (the accumulator is forwarded)
        operands = operands[1:3]
    elif not op.startswith(("ds_write", "global_store", "buffer_store", "scratch_store", "v_cmp")):
        operands = operands[1:]
    return set().union(*map(_registers, operands)) if operands else set()


def test_mfma_results_are_read_late_enough(kernels):
    """Along every way through the branches: the compiler counts along one of those that meet."""
    seen = set()
    for name, body in kernels.items():
        labels = {text[:-1]: i for i, text in enumerate(body) if text.endswith(":")}
        for i, text in enumerate(body):
            op = text.split()[0]
            if "mfma" not in op:
                continue
            seen.add(op)
            result = _registers(text.split(" ", 1)[1].split(",")[0])
            ways, least = [(i + 1, 0)], {}
            while ways:
                j, states = ways.pop()
                if j >= len(body) or states >= WAIT_STATES[op] or least.get(j, 99) <= states:
                    continue
                least[j] = states
                step = body[j]
                if step.endswith(":"):
                    ways.append((j + 1, states))
                    continue
                if step.startswith(("v_", "ds_", "global_", "buffer_", "scratch_", "flat_")):
                    assert not _read_by(step) & result, "%s: %s, %d wait states later %s" % (name, text, states, step)
                    if "mfma" in step and _registers(step.split(" ", 1)[1].split(",")[0]) == result:
                        continue                               # (the next one of the chain is looked at by itself)
                if step.startswith("s_endpgm"):
                    continue
                states += int(step.split()[1]) + 1 if step.startswith("s_nop") else 1
                if step.startswith(("s_branch", "s_cbranch")):
                    ways.append((labels[step.split()[1]], states))
                if not step.startswith("s_branch"):
                    ways.append((j + 1, states))
    assert "v_mfma_f32_32x32x16_bf16" in seen and len(seen) >= 3
