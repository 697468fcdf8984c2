"""CPU-only test of the built library's code: the wait states that matrix instructions need.

The product and convolution kernels issue v_mfma through inline assembly, where the compiler does not insert wait states: its code must not
touch an accumulator within seven states behind the instruction that writes it (a result of four passes), nor write an operand within
two states ahead of one that reads it, not even to move a value.  It did once, and the outputs were wrong."""
import concurrent.futures
import os
import re
import struct
import subprocess

import pytest

import paper_2507_11978_amd as nt

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
AFTER, AHEAD = 7, 2
REG = re.compile(r"\b([av])(?:\[(\d+):(\d+)\]|(\d+)\b)")


def code_objects(path):
    """The gfx950 images of the library's offload bundles."""
    data, magic, at, out = open(path, "rb").read(), b"__CLANG_OFFLOAD_BUNDLE__", 0, []
    while (at := data.find(magic, at)) >= 0:
        (count,), p = struct.unpack_from("<Q", data, at + len(magic)), at + len(magic) + 8
        for _ in range(count):
            off, size, n = struct.unpack_from("<QQQ", data, p)
            if size and b"gfx950" in data[p + 24:p + 24 + n]:
                out.append(data[at + off:at + off + size])
            p += 24 + n
        at += len(magic)
    return out


def registers(text):
    """Bit mask of the vector (low half) and accumulator registers named in `text`."""
    mask = 0
    for kind, lo, hi, one in REG.findall(text):
        lo, hi = (int(lo), int(hi)) if lo else (int(one), int(one))
        mask |= ((1 << (hi - lo + 1)) - 1) << (lo + (512 if kind == "a" else 0))
    return mask


def walk(code, start, results, writes, steps, found):
    """Follow straight code from `start` for `steps` instructions; results / writes: [mask, states left, text]."""
    for i in range(start, min(start + steps, len(code))):
        op, args, _ = code[i]
        mfma = op.startswith("v_mfma")
        vector = op[:2] == "v_" or op.startswith(("ds_", "global_", "buffer_", "flat_", "scratch_"))
        dest, _, rest = args.partition(",") if not args.startswith(("a[", "v[")) else (lambda j: (args[:j + 1], "", args[j + 1:]))(args.index("]"))
        if mfma:
            reads = registers(rest)
            found += [(t, f"{op} {args}") for m, _, t in writes if m & reads]
        elif vector and results:
            used = registers(args)
            found += [(t, f"{op} {args}") for m, _, t in results if m & used]
        passed = int(args) + 1 if op == "s_nop" else 1
        results[:] = [[m, c - passed, t] for m, c, t in results if c > passed]
        writes[:] = [[m, c - passed, t] for m, c, t in writes if c > passed]
        if mfma:
            if op.startswith("v_mfma_f32_16x16x32"):
                results.append([registers(dest), AFTER, f"{op} {args}"])
        elif op[:2] == "v_":
            writes.append([registers(dest if not op.startswith("v_permlane32_swap") else args), AHEAD, f"{op} {args}"])
        yield i
        if op in ("s_branch", "s_endpgm"):
            results.clear()
            writes.clear()


def hazards(image, tmp):
    tmp.write_bytes(image)
    text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(tmp)], check=True, capture_output=True, text=True).stdout
    found = []
    for body in re.split(r"\n\n", text)[1:]:
        name, _, body = body.partition(">:\n")
        if "v_mfma_f32_16x16x32" not in body:
            continue
        code = []
        for line in body.splitlines():
            ins, _, note = line.partition("//")
            op, _, args = ins.strip().partition(" ")
            if note:                                       # (padding has none)
                code.append((op, args.strip(), note))
        address = {int(note.split(":")[0], 16): i for i, (_, _, note) in enumerate(code)}
        first = min(address)
        results, writes, bad = [], [], []
        for i in walk(code, 0, results, writes, len(code), bad):
            # (what is pending at a branch is pending at its target, too)
            if code[i][0].startswith(("s_cbranch", "s_branch")) and (results or writes):
                j = address.get(first + int(re.search(r"\+0x([0-9a-f]+)>", code[i][2])[1], 16))
                for _ in walk(code, j, [list(r) for r in results], [list(w) for w in writes], AFTER, bad):
                    pass
        found += [(name.split("<")[-1], *b) for b in bad]
    return found


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler")
def test_no_accumulator_is_touched_around_its_matrix_instructions(tmp_path):
    images = code_objects(nt.lib_path())
    assert len(images) > 40
    with concurrent.futures.ProcessPoolExecutor(8) as pool:
        for bad in pool.map(hazards, images, [tmp_path / f"{i}.o" for i in range(len(images))]):
            assert not bad, bad[:4]
