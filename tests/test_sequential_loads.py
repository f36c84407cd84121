"""Host-side check of the built persistent sequential kernel: what its workgroups hand each other is loaded at agent scope, in every variant.
A load without the scope may be served by the vector cache of its CU, which can still hold the word that the same slot had three uses
ago: not an empty word, so the wait would end with an old value.  The objects were compiled here; no GPU needed."""
import glob
import os
import re
import shutil
import subprocess

import pytest

LLVM = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    import paper_2505_24791_amd as sjd
    if not os.path.exists(sjd.LIB_PATH):
        from paper_2505_24791_amd import build
        build.build()
    d = tmp_path_factory.mktemp("objects")
    shutil.copy(sjd.LIB_PATH, d / "libsjd.so")
    subprocess.run([f"{LLVM}/llvm-objdump", "--offloading", "libsjd.so"], cwd=d, check=True, stdout=subprocess.DEVNULL)
    found = {}
    for obj in glob.glob(str(d / "*gfx950")):
        names = subprocess.run([f"{LLVM}/llvm-objdump", "-t", obj], check=True, stdout=subprocess.PIPE, text=True).stdout
        names = re.findall(r" F \.text\s+\S+ (?:\.\S+ )?(\S*seq_persistent_kernel\S*)", names)
        if names:
            text = subprocess.run([f"{LLVM}/llvm-objdump", "-d", "--no-show-raw-insn", "--disassemble-symbols=" + ",".join(names), obj], check=True,
                                  stdout=subprocess.PIPE, text=True).stdout
            for part in re.split(r"^[0-9a-f]+ <", text, flags=re.M)[1:]:
                found[part.split(">")[0]] = part
    return found


def _accesses(text, what):
    """(descriptor registers, instruction) of each buffer access"""
    return [(re.search(r"s\[\d+:\d+\]", a).group(0), a) for a in re.findall(what + r" [^/\n]*", text)]


def test_exchanged_words_are_loaded_at_agent_scope(kernels):
    """All buffer stores go to the workspace that is exchanged, so their descriptor tells its loads from those of biases and cached rows."""
    assert len(kernels) >= 2 * 15                     # both 16-bit types
    for name, text in kernels.items():
        (ws,) = {d for d, _ in _accesses(text, r"buffer_store_dword(?:x\d)?")}
        loads = [a for d, a in _accesses(text, r"buffer_load_dwordx4") if d == ws]
        assert len(loads) >= 10, name
        assert all("sc1" in a for a in loads), (name, [a for a in loads if "sc1" not in a][:3])


def test_only_groups_of_one_xcd_store_to_their_own_l2(kernels):
    """The last template argument says that a group is one XCD; its results may stay in that XCD's L2, those of larger groups may not."""
    seen = set()
    for name, text in kernels.items():
        one = re.search(r"Lb[01]ELb([01])EE", name).group(1) == "1"
        seen.add(one)
        stores = _accesses(text, r"buffer_store_dword(?:x\d)?")
        assert len(stores) >= 10, name
        assert all(("sc1" in a) != one for _, a in stores), name
    assert seen == {True, False}


def test_every_launch_has_a_kernel_and_every_kernel_a_launch(kernels, launch_rules):
    """The variants (row blocks, width / 256, column blocks a round, cached rows ahead, one XCD) that the launch rules ask for, on any number of
    workgroups that can be set."""
    asked = set()
    for S in (1, 2, 3, 4):
        for n_cus in range(32, 257, 32):
            for batch in range(1, 257):
                xpg = launch_rules.xcds_per_group_on(256 * S, batch, n_cus)
                mb, per = 1 if batch <= 128 else 2, -(-64 * S // (n_cus // 8 * xpg))
                cb = 4 if mb == 2 or per > 2 else 2 if xpg == 1 and per < 2 else per      # as in launch_seq_persistent
                for tokens in (2, 256, 513, 600, 1024, 4096):
                    asked.add((mb, S, cb, launch_rules.rows_ahead(batch, 4 * S, 256 * S, tokens, n_cus, xpg), int(xpg == 1)))
    for mangled in ("DF16b", "DF16_"):
        built = {tuple(map(int, re.search(r"Li(\d)ELi(\d)ELi(\d)ELb([01])ELb([01])EE", k).groups())) for k in kernels if mangled in k}
        assert built == asked
