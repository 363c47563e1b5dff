"""What the compiler made of kernels whose speed hangs on it, read from the built library (no GPU)."""
import os
import re
import subprocess

import pytest

import paper_2605_26646_amd as umas

LLVM = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def code_objects(tmp_path_factory):
    """Paths of the code objects that the library holds, one per source."""
    if not os.path.exists(umas.lib_path()):
        import __graft_entry__ as g
        g.build()
    at = tmp_path_factory.mktemp("code")
    subprocess.run([f"{LLVM}/llvm-objcopy", "--dump-section", f".hip_fatbin={at}/bundles", umas.lib_path(), os.devnull], check=True)
    data = open(at / "bundles", "rb").read()
    paths, starts = [], [m.start() for m in re.finditer(b"\x7fELF", data)]
    for k, a in enumerate(starts):
        paths.append(str(at / f"{k}.o"))
        with open(paths[-1], "wb") as f:
            f.write(data[a:starts[k + 1] if k + 1 < len(starts) else len(data)])
    assert paths
    return paths


@pytest.fixture(scope="module")
def scratch(code_objects):
    """Bytes of scratch a lane takes, by kernel."""
    found = {}
    for path in code_objects:
        notes = subprocess.run([f"{LLVM}/llvm-readelf", "--notes", path], check=True, capture_output=True, text=True).stdout
        for kernel in notes.split("- .agpr_count:")[1:]:
            name = re.search(r"\.name:\s+(\S+)", kernel).group(1)
            found[name] = int(re.search(r"\.private_segment_fixed_size:\s+(\d+)", kernel).group(1))
    plain = subprocess.run(["c++filt"], input="\n".join(found), check=True, capture_output=True, text=True).stdout.split("\n")
    return {p.replace("umas::(anonymous namespace)::", "").removeprefix("void ").split("(")[0]: v for p, v in zip(plain, found.values())}


# sixteen bf16 vectors a lane fill the 512 registers of a wavefront to a few; no other instance has a reason to spill
def test_critic_rows_stay_in_registers(scratch):
    rows = {k: v for k, v in scratch.items() if k.startswith("k_value_rows<")}
    assert len(rows) == 2 * 5 * 4
    for name, size in rows.items():
        assert size <= (64 if name.startswith("k_value_rows<unsigned short, 16,") else 0), (name, size)


# the accumulators of a tile are half of its registers; who clears the taken tokens' entries must not keep them for that
def test_flagged_blocks_spill_little(scratch):
    assert scratch["k_dz_flagged"] <= 32


@pytest.fixture(scope="module")
def token_kernels(code_objects):
    """The instructions of the two routing kernels that write the per-token outputs: {stores past the caches or not: text}."""
    found = {}
    for path in code_objects:
        text = subprocess.run([f"{LLVM}/llvm-objdump", "-d", "--no-show-raw-insn", path], check=True, capture_output=True, text=True).stdout
        for past, body in re.findall(r"<\w*k_tokensILb([01])E\w*>:\n(.*?)(?=\n\n|\Z)", text, re.S):
            found[past == "1"] = body
    return found


# source index (two), turn and role of four tokens, where a wavefront's tokens are one segment's a lane and where they are not, in four rounds: stores that a
# compiler would make one with the plain ones of the paths beside them, and plain
def test_routing_stores_past_the_caches(token_kernels):
    past = re.compile(r"global_store_dwordx4 .* nt\b")
    assert len(past.findall(token_kernels[True])) == 4 * 2 * 4
    assert not past.findall(token_kernels[False])
