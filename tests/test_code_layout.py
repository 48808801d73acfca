"""Where the functions of a layer's kernel lie in the built library: a kernel directly behind the tile stages that it calls, so that a
call of one layer fetches its code, cold behind the weights of the call before, from one stretch of memory; every function at the start of
a cache line, so that code elsewhere does not move it against the lines."""
import re
import struct
import subprocess

from paper_2605_00686_amd import binding as B


def device_functions():
    """(address, size, demangled name) of the functions in the library's gfx950 code object, in address order."""
    data = open(B.LIB_PATH, "rb").read()
    at = data.index(b"__CLANG_OFFLOAD_BUNDLE__")
    n, pos = struct.unpack_from("<Q", data, at + 24)[0], at + 32
    code = b""
    for _ in range(n):
        offset, size, length = struct.unpack_from("<QQQ", data, pos)
        if b"gfx950" in data[pos + 24:pos + 24 + length]:
            code = data[at + offset:at + offset + size]
        pos += 24 + length
    assert code[:4] == b"\x7fELF"
    sh_off, = struct.unpack_from("<Q", code, 0x28)
    sh_size, sh_num = struct.unpack_from("<HH", code, 0x3A)
    sections = [struct.unpack_from("<IIQQQQIIQQ", code, sh_off + i * sh_size) for i in range(sh_num)]
    found = {}
    for _, kind, _, _, off, size, link, _, _, each in sections:
        if kind != 2:  # the symbol table
            continue
        names = sections[link][4]
        for i in range(size // each):
            name, info, _, _, value, length = struct.unpack_from("<IBBHQQ", code, off + i * each)
            if info & 15 == 2:  # a function
                text = code[names + name:code.index(b"\0", names + name)].decode()
                found[value] = (length, text)
    plain = subprocess.run(["c++filt"], input="\n".join(v[1] for v in found.values()), capture_output=True, text=True, check=True)
    return sorted((a, v[0], t) for (a, v), t in zip(found.items(), plain.stdout.splitlines()))


def test_a_kernel_lies_behind_its_stages():
    fns = device_functions()
    kernels = [i for i, f in enumerate(fns) if "moe::k_megakernel<" in f[2]]
    assert len(kernels) == 6
    for i in kernels:
        before, size, name = fns[i - 1]
        assert "tile_stage<" in name or "fused_stage<" in name, (fns[i][2], name)
        assert fns[i][0] - (before + size) < 256, fns[i][2]  # (kernels start on 256 bytes)
        assert re.search(r"\w+Policy(<moe::TileCfg<[^>]*>)?", name).group(0) in fns[i][2], (fns[i][2], name)


def test_functions_start_on_a_cache_line():
    assert all(address % 128 == 0 for address, _, name in device_functions() if "moe::" in name)
