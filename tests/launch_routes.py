"""Which kernels a call launches, found without a GPU: the runtime's launch calls are answered by the stand-in of test_launches.py, in a process of its own."""
import json
import os
import re
import subprocess
import sys

from test_launches import ROOT, STAND_IN

NOTING = STAND_IN.replace("#include <cstddef>", "#include <cxxabi.h>\n#include <cstdlib>\n#include <cstddef>").replace("    ++total;\n", r"""    ++total;
    char* name = abi::__cxa_demangle(names[kernel].c_str(), nullptr, nullptr, nullptr);
    printf("%u %s\n", config.grid.x * config.grid.y * config.grid.z, name ? name : names[kernel].c_str());
    free(name);
""")

CALLS = r"""
import ctypes, json, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)             # before the library: its calls are looked up here first
sys.path.insert(0, sys.argv[2])
import paper_2406_10181_amd as L
libc = ctypes.CDLL(None)
fake, big, code = 0x1000, 1 << 40, {"f32": 0, "f16": 1, "bf16": 2}
for what, shapes, r, d, dtype in json.loads(sys.argv[3]):
    m, n = shapes[0]
    if what == "compress":
        items = [(fake, fake, fake * (k + 1), fake * (k + 1), big, m, n) for k, (m, n) in enumerate(shapes)]
        L.lsp_compress_planned_grouped(L.compress_items(items), len(items), r, d, code[dtype], None)
    elif what == "apply":
        items = [(fake * (k + 1), fake, fake, fake, fake, fake, m, n) for k, (m, n) in enumerate(shapes)]
        L.lsp_decompress_apply_grouped(L.apply_items(items), len(items), r, d, code[dtype], None)
    else:
        L.lsp_estimation_bias(fake, fake, fake, fake, fake, fake, m, n, r, d, fake, fake, big, code[dtype])
    libc.printf(b"--\n")
libc.fflush(None)
"""


def launches(calls, where):
    """calls: (what, [(m, n), ...], r, d, dtype), what one of compress, apply, bias; where: a folder to work in.  For each a list of (kernel, workgroups)."""
    src, so = os.path.join(where, "noting.cpp"), os.path.join(where, "noting.so")
    with open(src, "w") as f:
        f.write(NOTING)
    subprocess.run([os.environ.get("CXX", "g++"), "-O1", "-std=c++17", "-shared", "-fPIC", src, "-o", so], check=True)
    out = subprocess.run([sys.executable, "-c", CALLS, so, ROOT, json.dumps(calls)], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, (out.returncode, out.stdout[-2000:], out.stderr[-2000:])
    found, now = [], []
    for line in out.stdout.splitlines():
        if line == "--":
            found.append(now)
            now = []
            continue
        grid, name = line.split(" ", 1)
        kernel = re.sub(r"\(lsp::WideForm\)|lsp::|^void ", "", name)
        now.append((kernel[: kernel.rindex("(")].replace("void ", ""), int(grid)))
    return found
