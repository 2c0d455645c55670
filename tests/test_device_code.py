"""CPU tests of the gfx950 code in libsc.so, disassembled: hazards that the hardware does not resolve and
that the compiler cannot see inside inline assembly."""
import os
import re
import struct
import subprocess

import pytest

from paper_2402_07710_amd import binding, build

OBJDUMP = os.path.join(os.path.dirname(os.path.dirname(build.HIPCC)), "llvm", "bin", "llvm-objdump")


@pytest.fixture(scope="module")
def instructions(tmp_path_factory):
    """The instructions of each gfx950 code object, in order."""
    binding.load()
    data = open(binding.LIB_PATH, "rb").read()
    out = []
    for at in (m.start() for m in re.finditer(re.escape(b"__CLANG_OFFLOAD_BUNDLE__"), data)):
        count, pos = struct.unpack_from("<Q", data, at + 24)[0], at + 32
        for _ in range(count):
            offset, size, name_len = struct.unpack_from("<QQQ", data, pos)
            target = data[pos + 24:pos + 24 + name_len]
            pos += 24 + name_len
            if b"gfx950" not in target:
                continue
            path = tmp_path_factory.mktemp("code") / "object.elf"
            path.write_bytes(data[at + offset:at + offset + size])
            text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(path)], capture_output=True, text=True, check=True).stdout
            out.append([line.split("//")[0].strip() for line in text.splitlines() if line.startswith("\t")])
    return out


def test_a_wait_state_between_writing_m0_and_a_load_to_lds(instructions):
    """A load into LDS takes its LDS address from M0; after a scalar write of M0 it needs one wait state (any
    instruction in between, s_nop 0 at least), or it may use the old address."""
    sites, bad = 0, []
    for code in instructions:
        for before, here in zip(code, code[1:]):
            mnemonic = here.split()[0]
            if "_load_lds_" in mnemonic or (mnemonic.startswith("buffer_load") and here.split()[-1] == "lds"):
                sites += 1
                if re.match(r"s_\w+ m0\b", before) or re.match(r"v_read(first)?lane_b32 m0\b", before):
                    bad.append((before, here))
    assert sites > 0
    assert not bad, f"{len(bad)} of {sites} loads into LDS directly behind a write of M0, e.g. {bad[0]}"


def test_steps_longer_than_the_list_of_offsets_allows_do_not_compile(tmp_path):
    """The general kernel reads its list of offsets two steps ahead; past the zeros behind the last offset it would gather at
    offsets that are none.  With fewer zeros than its longest step needs it must be refused."""
    path = os.path.join(build.CSRC, "sc_conv_gather.hip")
    text = open(path).read()
    zeros = re.search(r"LIST_PAD = (\d+);", text)
    short = tmp_path / "sc_conv_gather.hip"
    short.write_text(text.replace(zeros.group(0), f"LIST_PAD = {int(zeros.group(1)) - 1};"))
    run = subprocess.run([build.HIPCC, *build.FLAGS, "--cuda-device-only", "-fsyntax-only", str(short)], capture_output=True, text=True)
    assert run.returncode != 0 and "static assertion failed" in run.stderr and "the list's zeros reach" in run.stderr, run.stderr[-2000:]
