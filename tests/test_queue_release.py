"""The tile runs of the repair queue write subbins that a worker on another XCD
reads next, so every wave has to wait for its own stores before the barrier
after which one thread lets the tile go.  Checked on the built device code: on
no path from an agent-scope store of repair_run does a barrier or the function's
end come before a wait for all of the wave's vector memory operations."""
import os
import re
import subprocess

import pytest

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


@pytest.fixture(scope="module")
def functions(tmp_path_factory):
    if not os.path.exists(OBJDUMP):
        pytest.skip("llvm-objdump not available")
    from paper_2603_26968_amd import lopc
    d = tmp_path_factory.mktemp("dis")
    lib = str(d / "liblopc.so")
    os.symlink(lopc.LIB_PATH, lib)
    subprocess.run([OBJDUMP, "--offloading", lib], check=True, capture_output=True, cwd=d)
    out = {}
    for f in sorted(os.listdir(d)):
        if "gfx950" not in f:
            continue
        text = subprocess.run([OBJDUMP, "-d", str(d / f)], check=True, capture_output=True,
                              text=True).stdout
        name = None
        for line in text.splitlines():
            m = re.match(r"[0-9a-f]+ <(.*)>:$", line)
            if m:
                name = m.group(1)
            elif name and "repair_run" in name and re.match(r"\t[a-z]", line):
                m = re.match(r"\t(.*?)\s*// ([0-9A-F]+): (.*)$", line)
                out.setdefault(name, []).append((int(m.group(2), 16), m.group(1), m.group(3)))
    return out


def test_stores_are_waited_for_before_a_run_ends(functions):
    functions = {n: f for n, f in functions.items() if "batch_repair_run" not in n}
    assert len(functions) == 5, sorted(functions)  # one per tile shape
    for name, code in functions.items():
        at = {a: i for i, (a, _, _) in enumerate(code)}
        base = code[0][0]

        def successors(i):
            _, op, rest = code[i]
            m = re.match(r"s_(c?)branch", op)
            if not m:
                return [i + 1]
            t = re.search(r"<.*?\+0x([0-9a-f]+)>", rest)
            to = at[base + (int(t.group(1), 16) if t else 0)]
            return [to, i + 1] if m.group(1) else [to]

        stores = [i for i, (_, op, _) in enumerate(code) if re.match(r"(flat|global)_store.* sc1", op)]
        assert stores, name
        todo, seen = [s for i in stores for s in successors(i)], set()
        while todo:
            i = todo.pop()
            if i in seen:
                continue
            seen.add(i)
            op = code[i][1]
            if op.startswith("s_waitcnt") and "vmcnt(0)" in op:
                continue
            assert not re.match(r"s_(barrier|setpc|endpgm)", op), \
                f"{name}: {op} at {code[i][0]:x} with a store in flight"
            todo += successors(i)
