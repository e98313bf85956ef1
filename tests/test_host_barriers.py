"""Every workgroup barrier of the compiled kernels is reached with the wave's LDS operations waited for.  The compiler can leave the wait out
of a barrier at the head of a loop whose first trip has nothing to wait for; waves then read what others are still writing, now and then.
The built objects are disassembled and the LDS operations that may be outstanding followed through each kernel's flow."""
import re
import shutil
import subprocess

import pytest

LLVM = "/opt/rocm/llvm/bin"


def blocks_of(listing):
    """[(instructions, successors)] of one kernel's lines `address, text, branch target or None`; block 0 is the entry."""
    targets = {t for _, _, t in listing if t is not None}
    starts, fresh = [], True
    for i, (at, text, _) in enumerate(listing):
        if fresh or at in targets:
            starts.append(i)
        fresh = text.startswith(("s_cbranch", "s_branch", "s_endpgm", "s_setpc"))
    index = {listing[i][0]: b for b, i in enumerate(starts)}
    out = []
    for b, i in enumerate(starts):
        lines = listing[i:starts[b + 1] if b + 1 < len(starts) else len(listing)]
        _, text, target = lines[-1]
        after = [] if target is None else [index[target]]
        if not text.startswith(("s_branch", "s_endpgm", "s_setpc")) and b + 1 < len(starts):
            after.append(b + 1)
        out.append(([t for _, t, _ in lines], after))
    return out


def walk(state, instructions, found=None):
    """state: operations issued since the last LDS one that may be outstanding, or None.  LDS operations of a wave end in order."""
    for text in instructions:
        if text.startswith("s_waitcnt"):
            m = re.search(r"lgkmcnt\((\d+)\)", text)
            if m and state is not None and state >= int(m.group(1)):
                state = None
        elif text.startswith("ds_"):
            state = 0
        elif state is not None and text.startswith(("s_load", "s_buffer_load")):
            state += 1
        elif text.startswith("s_barrier") and found is not None and state is not None:
            found.append(text)
    return state


def unwaited_barriers(listing):
    blocks = blocks_of(listing)
    entry = [("unseen",)] * len(blocks)
    entry[0], work = None, [0]
    while work:
        b = work.pop()
        end = walk(entry[b], blocks[b][0])
        for s in blocks[b][1]:
            if entry[s] == ("unseen",):
                joined = end
            else:
                joined = min((x for x in (entry[s], end) if x is not None), default=None)
            if joined != entry[s]:
                entry[s] = joined
                work.append(s)
    found = []
    for b, (instructions, _) in enumerate(blocks):
        if entry[b] != ("unseen",):
            walk(entry[b], instructions, found)
    return len(found)


def kernels_of(text):
    """name -> listing, of llvm-objdump's output"""
    name, base, out = None, 0, {}
    for line in text.splitlines():
        m = re.match(r"([0-9a-f]+) <(\S+)>:", line)
        if m:
            base, name = int(m.group(1), 16), m.group(2)
            out[name] = []
            continue
        m = re.match(r"\s+(\S.*?)\s*// ([0-9A-F]+):", line)
        if m and name:
            t = re.search(r"<(\S+?)(?:\+0x([0-9a-f]+))?>$", line) if m.group(1).startswith(("s_cbranch", "s_branch")) else None
            out[name].append((int(m.group(2), 16), m.group(1), None if t is None else base + int(t.group(2) or "0", 16)))
    return {k: v for k, v in out.items() if any(t.startswith("s_barrier") for _, t, _ in v)}


def test_the_check_itself():
    waits = [(0, "ds_write_b32 v0, v1", None), (4, "s_waitcnt lgkmcnt(0)", None), (8, "s_barrier", None), (12, "ds_read_b32 v1, v0", None),
             (16, "s_waitcnt lgkmcnt(0)", None), (20, "ds_write_b32 v0, v1", None), (24, "s_cbranch_scc1 65530", 4), (28, "s_endpgm", None)]
    assert unwaited_barriers(waits) == 0
    assert unwaited_barriers([x for x in waits if x[0] != 4][:5] + [(24, "s_cbranch_scc1 65531", 8), (28, "s_endpgm", None)]) == 1
    early = [(0, "s_waitcnt lgkmcnt(0)", None)] + [(4 + a, t, g if g is None else 8 + 4) for a, t, g in waits[2:]]
    assert unwaited_barriers(early) == 1                     # the first trip has nothing outstanding, the second has


def disassembled(obj, where):
    subprocess.run([f"{LLVM}/llvm-objcopy", "--dump-section", f".hip_fatbin={where}/fatbin", str(obj), f"{where}/host.o"], check=True)
    subprocess.run([f"{LLVM}/clang-offload-bundler", "--unbundle", "--type=o", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", f"--input={where}/fatbin",
                    f"--output={where}/device.co"], check=True)
    return subprocess.run([f"{LLVM}/llvm-objdump", "-d", "--no-show-raw-insn", f"{where}/device.co"], check=True, capture_output=True, text=True).stdout


@pytest.mark.parametrize("source", ["hash_kernels", "score_kernels", "topk_kernels", "filter_kernels", "filter_groups"])
def test_no_barrier_leaves_lds_operations_behind(source, tmp_path):
    if shutil.which("hipcc") is None:
        pytest.skip("needs hipcc")
    from paper_2210_15748_amd import build as hip_build
    assert source + ".hip" in hip_build.SOURCES
    obj = hip_build.OBJ / (source + ".o")
    if not obj.exists() or hip_build.stale():
        hip_build.build(force=True)
    kernels = kernels_of(disassembled(obj, tmp_path))
    assert kernels
    bad = {k: n for k, v in kernels.items() if (n := unwaited_barriers(v))}
    assert not bad
