"""What the compiler makes of the device code, where correctness hangs on an instruction that no result shows reliably."""
import os
import re
import shutil
import subprocess

import pytest

import __graft_entry__ as build_entry

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def kernels(source, tmp_path):
    """Assembly of every function of a source file, by (mangled) name: lists of instructions and labels."""
    if not shutil.which(HIPCC):
        pytest.skip("no hipcc")
    out = tmp_path / "device.s"
    flags = build_entry.HIPCC_FLAGS + build_entry.PER_FILE_FLAGS.get(source, [])
    subprocess.run([HIPCC, *flags, "-x", "hip", "--offload-device-only", "-S", os.path.join(build_entry.CSRC, source), "-o",
                    str(out)], check=True, stderr=subprocess.DEVNULL)
    found, body = {}, None
    for line in out.read_text().splitlines():
        line = line.split(";")[0].strip()
        if re.match(r"_Z\w+:$", line):
            body = found.setdefault(line[:-1], [])
        elif line.startswith(".Lfunc_end"):
            body = None
        elif body is not None and line and (not line.startswith(".") or line.startswith(".LBB")):
            body.append(line)
    return found


def test_stores_are_complete_before_a_ticket_is_taken(tmp_path):
    """Workgroups that hand their results to the one that takes the last ticket: a barrier alone leaves stores of the other
    wavefronts in flight, so each wavefront has to wait for its own (vmcnt counts stores) right before the barrier."""
    seen = 0
    for name, body in kernels("retrieve.hip", tmp_path).items():
        if not re.search("retrieve_chunk_kernel|qrep_partial_kernel", name):
            continue
        tickets = [i for i, x in enumerate(body) if x.startswith(("global_atomic_add ", "flat_atomic_add "))]
        assert len(tickets) == 1, name
        barrier = max(i for i in range(tickets[0]) if body[i].startswith("s_barrier"))
        block = []                                   # the instructions in front of the barrier, back to a label or branch
        for x in reversed(body[:barrier]):
            if x.startswith((".LBB", "s_cbranch", "s_branch")):
                break
            block.append(x)
        assert any(re.match(r"s_waitcnt .*vmcnt\(0\)", x) for x in block), f"{name}: {block[:8]}"
        seen += 1
    assert seen == 4                                 # both kernels, both element types


def resources(source, tmp_path):
    """Bytes of private memory and of LDS of every kernel of a source file, from the metadata the compiler writes."""
    kernels(source, tmp_path)
    found = {}
    for part in (tmp_path / "device.s").read_text().split(".amdhsa_kernel ")[1:]:
        value = lambda key: int(re.search(rf"\.amdhsa_{key} (\d+)", part).group(1))
        found[part.split()[0]] = (value("private_segment_fixed_size"), value("group_segment_fixed_size"))
    return found


def test_finishing_kernel_of_the_percentile_shares_its_lds(tmp_path):
    """Its tile passes and its picks take turns: it needs the larger of the two (66 KB), not their sum (107 KB)."""
    got = {k: v for k, v in resources("seg.hip", tmp_path).items() if "quant_finish_kernel" in k}
    assert len(got) == 4 and all(lds <= 68 << 10 for _, lds in got.values()), got
