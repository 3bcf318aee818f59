"""How the update's workgroups hand their sums over, in the built code: on gfx950 a
store with sc1 has reached the memory that all XCDs share once vmcnt has counted it
down, so no counter may be advanced before that wait, and the reader has to drop its
own cached lines."""
import os

from paper_2511_19204_amd import build, hazards


def _kernels(part):
    out = {}
    for obj in hazards.code_objects(build.LIB):
        name = None
        for line in hazards.disassemble(obj).splitlines():
            if line.endswith(">:"):
                label = line.split("<")[1][:-2]
                if not (label.startswith("L") and label[1:].isdigit()):
                    name = label if part in label else None
                    if name:
                        out[name] = []
            elif name and line.startswith("\t"):
                out[name].append(line.split("//")[0].strip())
    return out


def test_sums_are_in_memory_before_they_are_counted():
    assert os.path.exists(build.LIB), "build the library first"
    kernels = {k: v for k, v in _kernels("update").items() if any("_atomic_add" in ln for ln in v)}
    assert len(kernels) == 3, list(kernels)  # 64 and 256 threads, and the one of update_noalloc
    for name, code in kernels.items():
        through, counted, waited, dropped = 0, 0, True, False
        for ln in code:
            if ln.startswith(("global_store", "flat_store")) and "sc1" in ln:
                through += 1
                waited = False
            elif ln.startswith("s_waitcnt") and "vmcnt(0)" in ln:
                waited = True
            elif ln.startswith(("global_atomic_add", "flat_atomic_add")):
                counted += 1
                assert waited, f"{name}: {ln}"
            elif ln.startswith("buffer_inv") and "sc1" in ln and counted:
                dropped = True
        assert through > 0 and counted > 0 and dropped, (name, through, counted, dropped)
