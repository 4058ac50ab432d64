"""Hand-offs between workgroups in the compiled kernels: where one thread writes the caches back for its workgroup, every wave has waited for
its own stores first.  The write-back only covers what has reached the L2, and a barrier does not wait for stores, so this cannot be left to
the barrier in front of it.  Read from the assembly that the compiler makes of these sources; no GPU."""
import os
import re
import shutil
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_2605_02218_amd import build as B


def _assembly(path, out):
    subprocess.run([B._hipcc(), *B.FLAGS, "-S", "--cuda-device-only", path, "-o", out], check=True, stderr=subprocess.PIPE)
    with open(out) as f:
        return f.read().split("\n")


def unguarded_write_backs(lines):
    """(kernel, line) of the write-backs whose workgroup barrier does not stand right behind a wait for all stores."""
    bad, kernel, found = [], "?", 0
    for i, line in enumerate(lines):
        m = re.match(r"(_Z\w+):", line)
        kernel = m.group(1) if m else kernel
        if "buffer_wbl2" not in line:
            continue
        found += 1
        j = i
        while j >= 0 and "s_barrier" not in lines[j] and not re.match(r"_Z\w+:", lines[j]):
            j -= 1
        before = [x.split(";")[0].strip() for x in lines[max(0, j - 40):j]]
        before = [x for x in before if x and not x.endswith(":")]
        waits = [k for k, x in enumerate(before) if x.startswith("s_waitcnt") and "vmcnt(0)" in x]
        stores = [k for k, x in enumerate(before) if re.match(r"(global|flat|buffer|scratch)_(store|atomic)", x)]
        if "s_barrier" not in lines[j] or not waits or (stores and stores[-1] > waits[-1]):
            bad.append((kernel, i + 1))
    return bad, found


def test_the_check_sees_a_missing_wait():
    good = ["_Zk:", "global_store_dword v0, v1, s[0:1]", "s_waitcnt vmcnt(0) lgkmcnt(0)", "s_barrier", "s_and_saveexec_b64 s[0:1], vcc", "buffer_wbl2 sc1"]
    assert unguarded_write_backs(good) == ([], 1)
    assert unguarded_write_backs([x.replace("vmcnt(0) ", "") for x in good]) == ([("_Zk", 6)], 1)
    assert unguarded_write_backs(good[:1] + good[2:3] + good[1:2] + good[3:]) == ([("_Zk", 6)], 1)


@pytest.mark.skipif(not (os.path.exists(B._hipcc()) or shutil.which(B._hipcc())), reason="no hipcc")
def test_every_wave_waits_for_its_stores_in_front_of_a_write_back(tmp_path):
    # the sources of kernels whose workgroups hand one another plain stores
    users = [s for s in B.SOURCES if re.search(r"image_barrier_wait\(|__ATOMIC_RELEASE", open(os.path.join(B.CSRC, s)).read())]
    assert {"eigen.hip", "greedy.hip"} <= set(users)
    with ThreadPoolExecutor(4) as ex:
        asm = list(ex.map(lambda s: _assembly(os.path.join(B.CSRC, s), str(tmp_path / (s + ".s"))), users))
    results = [unguarded_write_backs(a) for a in asm]
    assert sum(n for _, n in results) >= 4
    assert {s: bad for s, (bad, _) in zip(users, results) if bad} == {}


@pytest.mark.skipif(not (os.path.exists(B._hipcc()) or shutil.which(B._hipcc())), reason="no hipcc")
def test_an_image_of_the_small_sign_iteration_is_an_eighth_of_the_device(tmp_path):
    """What the launcher asks the runtime for each form of the kernel (split.hip), from the registers and the LDS it was compiled to: a
    workgroup per 16 x 16 tile on and below the diagonal, 256 compute units of four SIMDs with 512 registers and 160 KB."""
    text = "\n".join(_assembly(os.path.join(B.CSRC, "split.hip"), str(tmp_path / "split.s")))
    forms = {}
    for kernel in re.findall(r"\.amdhsa_kernel (\S*sign_small_kernelILi\d\S*)(.*?)\.end_amdhsa_kernel", text, re.S):
        value = {k: int(re.search(r"\.amdhsa_%s (\d+)" % k, kernel[1]).group(1)) for k in ("next_free_vgpr", "group_segment_fixed_size")}
        forms[int(re.search(r"ILi(\d)", kernel[0]).group(1))] = value
    assert sorted(forms) == [1, 2, 3, 4]
    for blocks, v in forms.items():
        waves = 512 // ((v["next_free_vgpr"] + 7) // 8 * 8)                    # of a SIMD; a workgroup has one on each
        held = 256 * min(waves, 8, 160 * 1024 // v["group_segment_fixed_size"])
        tiles = 4 * blocks * (4 * blocks + 1) // 2
        assert tiles <= held // 8, (blocks, tiles, held)
