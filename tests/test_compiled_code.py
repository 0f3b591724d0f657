"""Waits in the built gfx950 code that the compiler does not insert: the wait states that statements of inline assembly
have to bring along, and what has to have arrived before a bare barrier.  Needs no GPU."""
import re
import shutil
import struct
import subprocess

import pytest

import paper_2604_10152_amd as sm
from paper_2604_10152_amd import binding

OBJDUMP = shutil.which("llvm-objdump", path="/opt/rocm/llvm/bin") or shutil.which("llvm-objdump")


def _code_objects():
    sm.load_library()                                       # builds it if it is not there
    blob, magic, at = open(binding.lib_path(), "rb").read(), b"__CLANG_OFFLOAD_BUNDLE__", 0
    while (at := blob.find(magic, at)) >= 0:
        p = at + len(magic)
        (entries,) = struct.unpack_from("<Q", blob, p)
        p += 8
        for _ in range(entries):
            offset, size, n = struct.unpack_from("<QQQ", blob, p)
            if b"gfx950" in blob[p + 24:p + 24 + n] and size:
                yield blob[at + offset:at + offset + size]
            p += 24 + n
        at += len(magic)


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """Every function as its instructions in order, each (address, text)."""
    if OBJDUMP is None:
        pytest.skip("no llvm-objdump")
    out = []
    for i, code in enumerate(_code_objects()):
        path = tmp_path_factory.mktemp("code") / f"{i}.co"
        path.write_bytes(code)
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", str(path)],
                              capture_output=True, text=True, check=True).stdout
        for line in text.splitlines():
            if line.endswith(">:"):
                out.append([])
            elif line.startswith("\t") and "//" in line:
                instruction, _, comment = line.partition("//")
                out[-1].append((int(comment.split(":")[0], 16), " ".join(instruction.split())))
    return out


@pytest.fixture(scope="module")
def listing(kernels):
    return [x for kernel in kernels for _, x in kernel]


def test_lds_loads_take_their_base_from_a_scalar_move(listing):
    """A load that reads a scalar register needs five wait states behind a vector instruction that wrote it
    (v_readlane of a spilled pointer); a scalar move right before it waits by itself."""
    at = [i for i, x in enumerate(listing) if x.startswith("global_load_lds_")]
    assert len(at) > 500
    for i in at:
        base = re.search(r"(s\[\d+:\d+\])", listing[i]).group(1)
        assert listing[i - 1].startswith(f"s_mov_b64 {base},"), listing[i - 6:i + 1]
        assert listing[i - 2].startswith("s_mov_b32 m0,"), listing[i - 6:i + 1]


def test_hinted_stores_keep_their_data_for_two_wait_states(listing):
    """A vector instruction must not write the data registers of a 16-byte store within two wait states behind it."""
    at = [i for i, x in enumerate(listing) if x.startswith("global_store_dwordx4") and x.endswith(" nt")]
    assert len(at) > 500
    for i in at:
        m = re.fullmatch(r"s_nop (\d+)", listing[i + 1])
        assert m and int(m.group(1)) >= 1, listing[i:i + 4]


def test_no_barrier_leaves_lds_writes_in_flight(kernels):
    """A barrier does not wait for the LDS writes of the wave that arrives there; what other waves read behind it has to
    be written before.  Followed along every branch."""
    barriers = 0
    for kernel in kernels:
        index = {address: i for i, (address, _) in enumerate(kernel)}
        pending = [False] * len(kernel)                     # LDS writes in flight in front of the instruction
        todo = [i for i, (_, x) in enumerate(kernel) if x.startswith("ds_write")]
        while todo:
            i = todo.pop()
            address, x = kernel[i]
            waits = x.startswith("s_waitcnt") and "lgkmcnt(0)" in x
            if not (pending[i] or x.startswith("ds_write")) or waits:
                continue
            after = [] if x.startswith(("s_branch", "s_endpgm")) else [i + 1]
            if x.startswith(("s_branch", "s_cbranch")):
                step = int(x.split()[1])
                after.append(index[address + 4 + 4 * (step - 65536 if step >= 32768 else step)])
            for j in after:
                if not pending[j]:
                    pending[j] = True
                    todo.append(j)
        for i, (_, x) in enumerate(kernel):
            if x.startswith("s_barrier"):
                barriers += 1
                assert not pending[i], kernel[max(0, i - 12):i + 1]
    assert barriers > 200
