"""What the compiler notes about the built kernels (the code objects inside libconef.so): argument bytes, registers, spills.  Costs that
no result shows, so a change that brings them back would pass every other test."""
import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_2312_08538_amd import binding as B

LLVM = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{demangled kernel name: {argument bytes, vector registers, spilled ones}}"""
    if not os.path.exists(f"{LLVM}/llvm-readelf") or shutil.which("c++filt") is None:
        pytest.skip("no binary tools")
    tmp = tmp_path_factory.mktemp("co")
    subprocess.run([f"{LLVM}/llvm-objcopy", "--dump-section", f".hip_fatbin={tmp}/fatbin", B.LIB_PATH, f"{tmp}/copy"], check=True)
    data, found, pos = (tmp / "fatbin").read_bytes(), {}, 0
    while (start := data.find(b"__CLANG_OFFLOAD_BUNDLE__", pos)) >= 0:
        count, at = struct.unpack_from("<Q", data, start + 24)[0], start + 32
        for _ in range(count):
            off, size, length = struct.unpack_from("<QQQ", data, at)
            target = data[at + 24:at + 24 + length].decode()
            at += 24 + length
            if "gfx950" not in target or size == 0:
                continue
            (tmp / "object").write_bytes(data[start + off:start + off + size])
            notes = subprocess.run([f"{LLVM}/llvm-readelf", "--notes", f"{tmp}/object"], check=True, capture_output=True, text=True).stdout
            for block in notes.split(".agpr_count:")[1:]:
                def number(key):
                    return int(re.search(rf"\.{key}:\s+(\d+)", block).group(1))
                # (the arguments that the compiler adds for itself come behind the declared ones)
                args = max((int(o) + int(n) for o, n, kind in re.findall(r"\.offset:\s+(\d+)\s+\.size:\s+(\d+)\s+\.value_kind:\s+(\w+)", block)
                            if not kind.startswith("hidden")), default=0)
                name = re.search(r"\.symbol:\s+'?([\w$.]+?)\.kd", block).group(1)
                found[name] = {"args": args, "vgprs": number("vgpr_count"), "spills": number("vgpr_spill_count")}
        pos = start + 32
    names = subprocess.run(["c++filt"], input="\n".join(found), check=True, capture_output=True, text=True).stdout.split("\n")
    out = {re.sub(r"^void |conef::\(anonymous namespace\)::|\(.*$", "", n.replace("(anonymous namespace)", "{}").replace("conef::{}::", "")): v
           for n, v in zip(names, found.values())}
    assert len(out) == len(found) > 100
    return out


def test_a_launch_carries_no_more_than_its_kernel_reads(kernels):
    """The plan that a kernel is given holds what kernels read (512 bytes at most), not what only launchers do: every line of 64
    bytes costs each launch time.  What else a kernel takes are a dozen pointers at the most."""
    assert max(k["args"] for k in kernels.values()) <= 512 + 128


def test_octet_q_pass_holds_two_steps_at_rank_8(kernels):
    """k_q_octet's waves load the next step's octets and rows of P^ while they work on this one.  At rank 8 that takes all the
    registers that its occupancy leaves (168 with fp32 gradients, 128 with bf16); far fewer mean that the compiler has put the loads behind
    the work, which costs a quarter of the pass."""
    for bits in (2, 4, 8):
        assert kernels[f"k_q_octet<false, {bits}, 2, false, 0>"]["vgprs"] > 144
        assert kernels[f"k_q_octet<true, {bits}, 2, false, 0>"]["vgprs"] > 112
