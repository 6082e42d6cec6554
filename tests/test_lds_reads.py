"""The device code of the GEMMs that was built: no instruction touches a register while an LDS read into it is under way.
Their K loops read fragments by inline assembly and wait for them by count, the tiles of one block to a wave across the
loop's end, where the compiler, which knows of no read under way, is free to copy a register. Such a copy would take the value
of before the read: wrong results that depend on timing. So every path through each kernel is followed here."""
import re
import subprocess

from test_store_instructions import gfx950_code_objects, objdump

# LDS operations end in order, so one with n newer ones has ended once at most n may be outstanding. Kept newest first, more than
# lgkmcnt (at most 15) can tell apart in one.
DEPTH = 17
HEAD = re.compile(r"^[0-9a-f]+ <(.+)>:$")
LINE = re.compile(r"^\s+(\S+)\s*(.*?)\s*//\s*([0-9A-F]+):.*?(?:<\S+?\+0x([0-9a-f]+)>)?$")
REGISTER = re.compile(r"\b([va])(?:(\d+)|\[(\d+):(\d+)\])")


def registers(operands):
    found = set()
    for kind, one, first, last in REGISTER.findall(operands):
        lo, hi = (int(one), int(one)) if one else (int(first), int(last))
        found |= {(kind, r) for r in range(lo, hi + 1)}
    return found


def kernels(listing):
    """{name: [(address from the start, mnemonic, operands, branch target or None)]} of a disassembly."""
    found, code, start = {}, None, None
    for line in listing:
        m = HEAD.match(line)
        if m:
            code = found[m.group(1)] = []
            start = None
            continue
        m = LINE.match(line)
        if not m or code is None:
            continue
        at = int(m.group(3), 16)
        start = at if start is None else start
        target = int(m.group(4), 16) if m.group(4) else (0 if line.rstrip().endswith(">") and "branch" in m.group(1) else None)
        code.append((at - start, m.group(1), m.group(2), target))
    return found


def reads_in_flight(code):
    """The instructions of a kernel that may touch a register with an LDS read into it under way, and how many reads it has."""
    index = {at: i for i, (at, *_) in enumerate(code)}
    starts = sorted({0} | {index[t] for _, _, _, t in code if t is not None} |
                    {i + 1 for i, c in enumerate(code) if c[3] is not None or c[1] == "s_endpgm"})
    blocks = {a: b for a, b in zip(starts, starts[1:] + [len(code)]) if a < len(code)}
    touched = [registers(ops) for _, _, ops, _ in code]
    pending, todo, bad, reads = {0: ()}, [0], set(), 0
    while todo:
        block = todo.pop()
        state, last = list(pending[block]), None
        for i in range(block, blocks[block]):
            _, op, ops, target = code[i]
            assert not op.startswith(("s_setpc", "s_swappc", "s_call")), op
            if any(touched[i] & into for into in state):
                bad.add(i)
            if op.startswith("ds_"):
                into = set() if op.startswith("ds_write") else registers(ops.split(",")[0])
                state.insert(0, frozenset(into))
                if len(state) > DEPTH:
                    state[DEPTH - 1:] = [frozenset().union(*state[DEPTH - 1:])]
            elif op == "s_waitcnt":
                m = re.search(r"lgkmcnt\((\d+)\)", ops)
                if m:
                    del state[int(m.group(1)):]
            last = (i, op, target)
        i, op, target = last
        follow = [] if op in ("s_endpgm", "s_branch") else [i + 1]
        follow += [index[target]] if target is not None else []
        for f in follow:
            old = pending.get(f)
            new = list(state) if old is None else [
                frozenset().union(*(s[k] for s in (old, state) if k < len(s))) for k in range(max(len(old), len(state)))]
            if old is None or tuple(new) != old:
                pending[f] = tuple(new)
                todo.append(f)
    return [" ".join(code[i][1:3]) for i in sorted(bad)], sum(op.startswith("ds_read") for _, op, _, _ in code)


def listing(*lines):
    """A disassembly of instructions of four bytes; "op operands -> n" branches to the n-th."""
    out = ["0000000000001000 <k>:"]
    for i, line in enumerate(lines):
        text, _, to = line.partition(" -> ")
        out.append("\t%s // %012X: BF800000%s" % (text, 0x1000 + 4 * i, " <k+0x%x>" % (4 * int(to)) if to else ""))
    return kernels(out)["k"]


def test_the_check_sees_what_it_should():
    loop = ["ds_read_b128 v[0:3], v9", "ds_read_b128 v[4:7], v9", "s_waitcnt lgkmcnt(1)", "v_mfma_f32 a[0:3], v[0:3], v[0:3], a[0:3]",
            "ds_read_b128 v[0:3], v9 offset:256", "s_waitcnt lgkmcnt(1)", "v_mfma_f32 a[0:3], v[4:7], v[4:7], a[0:3]",
            "ds_read_b128 v[4:7], v9 offset:512", "s_cbranch_scc1 65529 -> 2", "s_waitcnt lgkmcnt(0)", "s_endpgm"]
    assert reads_in_flight(listing(*loop)) == ([], 4)
    copied = loop[:8] + ["v_mov_b32_e32 v20, v5"] + loop[8:]                        # a copy at the loop's end
    assert reads_in_flight(listing(*copied)) == (["v_mov_b32_e32 v20, v5"], 4)
    late = loop[:5] + ["s_waitcnt lgkmcnt(2)"] + loop[6:]                           # waits for one read too few
    assert reads_in_flight(listing(*late)) == ([loop[6], loop[7]], 4)
    assert reads_in_flight(listing(*loop[:9] + ["v_add_u32 v1, v0, v9"] + loop[9:])) == (["v_add_u32 v1, v0, v9"], 4)
    assert reads_in_flight(listing("ds_read_b64 a[2:3], v0", "ds_write_b32 v0, v1", "s_waitcnt lgkmcnt(1)", "v_accvgpr_read_b32 v5, a3",
                                   "s_endpgm")) == ([], 1)
    assert reads_in_flight(listing("ds_read_b64 a[2:3], v0", "s_waitcnt vmcnt(0)", "v_accvgpr_read_b32 v5, a3", "s_endpgm"))[0] != []
    # on one of two paths only; further back than lgkmcnt counts
    assert reads_in_flight(listing("s_cbranch_scc0 1 -> 2", "ds_read_b32 v7, v0", "v_mov_b32_e32 v1, v7", "s_endpgm"))[0] == ["v_mov_b32_e32 v1, v7"]
    many = ["ds_read_b32 v%d, v0" % (10 + i) for i in range(30)]
    assert reads_in_flight(listing(*many, "s_waitcnt lgkmcnt(15)", "v_mov_b32_e32 v1, v24", "v_mov_b32_e32 v1, v25", "s_endpgm"))[0] == [
        "v_mov_b32_e32 v1, v25"]
    assert reads_in_flight(listing(*many, "v_mov_b32_e32 v1, v10", "s_endpgm"))[0] == ["v_mov_b32_e32 v1, v10"]


def test_no_register_is_used_with_an_lds_read_into_it_under_way(tmp_path):
    seen = {"gemm_tile_kernel": 0, "gemm_bf16_kernel": 0}
    for i, code_object in enumerate(gfx950_code_objects()):
        if not any(name.encode() in code_object for name in seen):
            continue
        path = tmp_path / ("%d.co" % i)
        path.write_bytes(code_object)
        p = subprocess.run([objdump(), "-d", "--mcpu=gfx950", str(path)], stdout=subprocess.PIPE, text=True, check=True)
        for name, code in kernels(p.stdout.splitlines()).items():
            kind = [k for k in seen if k in name]
            if kind:
                bad, reads = reads_in_flight(code)
                assert not bad, (name, bad[:5])
                assert reads > 4, name
                seen[kind[0]] += 1
    assert seen["gemm_tile_kernel"] > 30 and seen["gemm_bf16_kernel"] > 8, seen
