"""Order of LDS accesses in the compiled kernels, where no run would show a missing barrier.  The device code of the built library is taken
out of its offload bundles and its branches are followed; no GPU is needed."""
import re
import struct
import subprocess

import pytest

import paper_1911_10175_amd as st

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


def device_code(symbol, tmp_path):
    """The ELF of the bundle whose kernels' names contain `symbol`."""
    lib = open(st.lib_path(), "rb").read()
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = lib.find(magic)
    while at >= 0:
        count, p = struct.unpack_from("<Q", lib, at + 24)[0], at + 32
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", lib, p)
            blob = lib[at + offset:at + offset + size]
            p += 24 + length
            if symbol in blob:
                path = tmp_path / "device.elf"
                path.write_bytes(blob)
                return path
        at = lib.find(magic, at + 24)
    raise AssertionError("kernel not in the library")


def kernels(symbol, tmp_path):
    """{kernel: [(address, instruction, address it may branch to)]}"""
    text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(device_code(symbol.encode(), tmp_path))], check=True, capture_output=True, text=True).stdout
    found, start = {}, 0
    for line in text.splitlines():
        head = re.match(r"([0-9a-f]+) <(\S+)>:", line)
        if head:
            start, body = int(head[1], 16), found.setdefault(head[2], [])
        elif "//" in line and found:
            code, _, rest = line.partition("//")
            target = re.search(r"\+0x([0-9a-f]+)>", rest)
            body.append((int(rest.split(":")[0], 16), code.split()[0], start + int(target[1], 16) if target else None))
    return {k: v for k, v in found.items() if symbol in k}


def writes_without_barrier(body):
    """Addresses of single words written to LDS on a path on which tiles (8 bytes a lane) have been written since the last barrier."""
    index = {a: i for i, (a, _, _) in enumerate(body)}
    seen, bad, work = set(), set(), [(0, False)]
    while work:
        i, dirty = work.pop()
        while i < len(body) and (i, dirty) not in seen:
            seen.add((i, dirty))
            address, op, target = body[i]
            assert not op.startswith(("s_setpc", "s_swappc", "s_call")), "a jump that cannot be followed"
            if op.startswith("ds_write") and op.endswith("_b64"):
                dirty = True
            elif op.startswith("ds_write") and op.endswith("_b32") and dirty:
                bad.add(hex(address))
            elif op == "s_barrier":
                dirty = False
            elif op == "s_endpgm":
                break
            elif op.startswith(("s_branch", "s_cbranch")):
                work.append((index[target], dirty))
                if op == "s_branch":
                    break
            i += 1
    return bad


def test_counts_of_small_values_are_not_overwritten_by_tiles(tmp_path):
    """Filter gradients on f16 pieces: a wavefront's count lies where others may still write the halo of a tile.  Without a barrier before it
    the count is lost, and gradients that should have been computed again are not."""
    found = kernels("bww_dense_half_kernel", tmp_path)
    assert len(found) == 2, sorted(found)                       # two tile shapes
    for name, body in found.items():
        ops = [op for _, op, _ in body]
        assert any(op.startswith("ds_write") and op.endswith("_b64") for op in ops) and any(op.startswith("ds_write") and op.endswith("_b32") for op in ops), name
        assert not writes_without_barrier(body), f"{name}: {sorted(writes_without_barrier(body))}"


@pytest.mark.parametrize("ops,bad", [
    ("ds_write_b32 s_barrier ds_write2st64_b64 s_barrier ds_write_b32", 0), ("ds_write2st64_b64 ds_write_b32", 1), ("ds_write_b64 s_barrier s_endpgm ds_write_b32", 0)])
def test_the_check_sees_what_it_is_for(ops, bad):
    assert len(writes_without_barrier([(4 * i, op, None) for i, op in enumerate(ops.split())])) == bad


def test_the_check_follows_branches():
    loop = [(0, "ds_write_b32", None), (4, "s_barrier", None), (8, "ds_write2st64_b64", None), (12, "s_cbranch_scc1", 24), (16, "s_barrier", None),
            (20, "s_branch", 8), (24, "ds_write_b32", None), (28, "s_endpgm", None)]
    assert writes_without_barrier(loop) == {hex(24)}
