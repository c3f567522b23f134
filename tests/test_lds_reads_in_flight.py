"""LDS reads issued from inline assembly are in flight until the wait written for them, and the compiler does not know: a copy or a
spill it puts in between moves a value that has not arrived.  The built library's own gfx950 code is walked along every path: no
instruction touches a register whose LDS read nobody has waited for, and where the pipelined loop (K and V operands of several
matrix instructions in flight at once) leaves its straight line, the way it takes waits for them first."""
import os
import re
import struct
import subprocess

import pytest

from paper_2510_26577_amd import binding

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
REGISTERS = re.compile(r"\b([va])(?:(\d+)|\[(\d+):(\d+)\])")
LINE = re.compile(r"^\t(\S+)\s*(.*?)\s*// ([0-9A-F]+): .*?(?:\+0x([0-9a-f]+)>)?$")
HEAD = re.compile(r"^([0-9a-f]+) <(.+)>:$")


def registers(text):
    out = set()
    for kind, one, first, last in REGISTERS.findall(text):
        out.update((kind, i) for i in range(int(one or first), int(one or last) + 1))
    return out


def parse(listing):
    """{kernel: [(operation, operands, index of the branch's target or None)]}"""
    found, base, rows = {}, 0, None
    for line in listing.splitlines():
        if m := HEAD.match(line):
            base, rows = int(m[1], 16), found.setdefault(m[2], [])
        elif rows is not None and (m := LINE.match(line)):
            rows.append((int(m[3], 16) - base, m[1], m[2], int(m[4], 16) if m[4] else 0))
    out = {}
    for name, rows in found.items():
        at = {r[0]: i for i, r in enumerate(rows)}
        out[name] = [(op, args, at[to] if op.startswith(("s_cbranch", "s_branch")) else None) for _, op, args, to in rows]
    return out


def follow(code, i):
    op, _, to = code[i]
    ways = [] if to is None else [to]
    return ways if op in ("s_branch", "s_endpgm", "s_setpc_b64") or i + 1 == len(code) else ways + [i + 1]


def lgkm_wait(code, i):
    """How many operations the wait at i leaves outstanding; None: not a wait for LDS."""
    m = re.search(r"lgkmcnt\((\d+)\)", code[i][1]) if code[i][0] == "s_waitcnt" else None
    return int(m[1]) if m else None


def in_flight(code, reads=r"ds_(read|bpermute|permute|swizzle)"):
    """Per instruction: {register: LDS operations issued after its read}, the fewest over all ways there (LDS answers in order,
    so a wait that leaves n outstanding has seen every read with n or more behind it).  And the instructions that touch one."""
    state, touched, work = [None] * len(code), set(), [0]
    state[0] = {}
    used = [registers(args) for _, args, _ in code]
    while work:
        i = work.pop()
        op, args, _ = code[i]
        now = dict(state[i])
        left = lgkm_wait(code, i)
        if left is not None:
            now = {r: n for r, n in now.items() if n < left}
        elif op != "s_waitcnt":
            if used[i] & now.keys():
                touched.add(i)
            if op.startswith("ds_"):
                now = {r: n + 1 for r, n in now.items()}
                if re.match(reads, op):
                    now.update((r, 0) for r in registers(args.split(",")[0]))
        for s in follow(code, i):
            old = state[s]
            new = now if old is None else {r: min(old.get(r, 99), now.get(r, 99)) for r in old.keys() | now.keys()}
            new = {r: min(n, 16) for r, n in new.items()}  # (the counter holds 4 bits)
            if new != old:
                state[s] = new
                work.append(s)
    return [s or {} for s in state], touched


def waits_first(code, i):
    while lgkm_wait(code, i) is None:
        if code[i][0] == "s_branch":
            i = code[i][2]
        elif code[i][2] is not None or code[i][0] == "s_endpgm":
            return False
        else:
            i += 1
    return True


def listing_of(lines):
    """A listing in the disassembler's form: every line an instruction of 4 bytes; a branch names its target's line."""
    out = ["0000000000001000 <k>:"]
    for i, line in enumerate(lines):
        m = re.match(r"(s_c?branch\S*) (\d+)$", line)
        text, to = (m[1] + " 0", f" <k+0x{4 * int(m[2]):x}>") if m and int(m[2]) else (line, "")
        out.append(f"\t{text} // {0x1000 + 4 * i:012X}: 00000000{to}")
    return "\n".join(out)


READ, USE, COPY, DONE = "ds_read_b128 v[0:3], v9", "v_add_f32_e32 v8, v1, v1", "v_mov_b32_e32 v7, v2", "s_endpgm"


@pytest.mark.parametrize("lines, want", [
    ([READ, "s_waitcnt lgkmcnt(0)", USE, DONE], []),
    ([READ, USE, DONE], [1]),
    ([READ, COPY, "s_waitcnt lgkmcnt(0)", USE, DONE], [1]),
    ([READ, "ds_read_b64 v[10:11], v9", "s_waitcnt lgkmcnt(1)", USE, DONE], []),
    ([READ, "ds_read_b64 v[10:11], v9", "s_waitcnt lgkmcnt(1)", "v_mov_b32_e32 v7, v11", DONE], [3]),
    ([READ, "s_waitcnt vmcnt(0)", USE, DONE], [2]),
    # over a loop's back edge, and on one of two ways
    ([COPY, READ, "s_cbranch_scc1 4", "s_waitcnt lgkmcnt(0)", "s_branch 6", DONE, "s_cbranch_scc0 1", DONE], [1]),
    (["s_cbranch_vccz 2", READ, "s_waitcnt vmcnt(0)", USE, DONE], [3]),
])
def test_the_walk_finds_registers_touched_too_early(lines, want):
    assert sorted(in_flight(parse(listing_of(lines))["k"])[1]) == want


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    if not os.path.exists(binding.LIB_PATH):
        binding.build_library()
    data = open(binding.LIB_PATH, "rb").read()
    found, at, folder = {}, 0, tmp_path_factory.mktemp("code")
    while (at := data.find(b"\x7fELF\x02\x01\x01\x40", at)) >= 0:  # 64-bit little-endian, OS/ABI AMDGPU_HSA
        shoff, = struct.unpack_from("<Q", data, at + 40)
        shentsize, shnum = struct.unpack_from("<HH", data, at + 58)
        path = folder / f"{at}.co"
        path.write_bytes(data[at:at + shoff + shentsize * shnum])
        found.update(parse(subprocess.run([OBJDUMP, "-d", "--mcpu=gfx950", str(path)], capture_output=True, text=True, check=True).stdout))
        at += 64
    assert sum("attn_kernel" in n for n in found) >= 28
    return found


def test_no_kernel_touches_a_register_whose_read_is_in_flight(kernels):
    for name, code in kernels.items():
        touched = in_flight(code)[1]
        assert not touched, (name, [code[i][:2] for i in sorted(touched)][:4])


@pytest.mark.parametrize("shape", ["8ELi1ELi1ELb0", "8ELi1ELi1ELb1", "4ELi2ELi1ELb0", "2ELi2ELi1ELb0"])
def test_the_pipelined_loop_waits_for_its_reads_wherever_it_is_left(kernels, shape):
    """The 256-row shape with D = 128 and 16-bit K/V, dense and paged, the 128-row and the deep 64-row shape dense: 24 to 32 registers of
    operands of both products are in flight there; the branches of a tile's barrier meet 16, others reads of one kind."""
    (name, code), = [(n, c) for n, c in kernels.items() if f"attn_kernelILi128ELi{shape}ELi4ELb0E" in n]
    state, of_v = in_flight(code)[0], in_flight(code, r"ds_read_b64_tr_b16")[0]
    seen = 0
    for i, (op, _, to) in enumerate(code):
        if op.startswith("s_cbranch") and len(state[i]) >= 24 and of_v[i]:
            assert waits_first(code, to), (name, code[i], to)
            seen += 1
    assert seen >= 4, seen  # out of the blocks of the first tile and of the loops'


@pytest.mark.parametrize("shape, loads", [("4ELi2ELi1ELb0", 4), ("2ELi2ELi1ELb0", 8)])
def test_the_pipelined_loops_of_two_key_groups_keep_three_tiles_in_flight(kernels, shape, loads):
    """As the plain loop does (`loads` of a wave to a tile of K and V): at a barrier behind which a full tile is queued, those of the two
    tiles before it may be outstanding."""
    (name, code), = [(n, c) for n, c in kernels.items() if f"attn_kernelILi128ELi{shape}ELi4ELb0E" in n]
    allowed = []
    for i, (op, _, _) in enumerate(code):
        if op != "s_barrier":
            continue
        queued, j = 0, i + 1
        while not code[j][0].startswith(("s_cbranch", "s_branch", "s_barrier", "s_endpgm")):
            queued += code[j][0] == "global_load_lds_dwordx4"
            j += 1
        if queued == loads:
            allowed += [int(m[1]) for o, a, _ in code[i - 3:i] if o == "s_waitcnt" and (m := re.search(r"vmcnt\((\d+)\)", a))][-1:]
    assert len(allowed) >= 5 and set(allowed) == {2 * loads}, (name, allowed)
