"""Code generation of the any-N kernel (CPU only, cross-compiled for gfx950):
everything in registers but the write-back stash, which takes the same share
of the compute unit's LDS as in the fixed-N kernels; non-temporal gradient
loads; no atomics."""

import re

from paper_1805_07891_amd import build


def test_any_n_kernels(tmp_path):
    out = tmp_path / "fused_many.s"
    asm = open(build.device_assembly(str(out), "fused_many.hip")).read()
    seen = set()
    for block in asm.split("  - .agpr_count:")[1:]:
        name = re.search(r"\.name:\s+(\S+)", block).group(1)
        opt = int(re.search(r"fused_step_manyILi(\d)E", name).group(1))
        seen.add(opt)

        def field(key):
            return int(re.search(rf"\.{key}:\s+(\d+)", block).group(1))

        states = {0: 2, 1: 2, 2: 1, 3: 3}[opt]
        tiles = (40 * 1024) // (states * 4 * 1024)
        assert field("group_segment_fixed_size") == 4 * tiles * states * 4 * 1024, name
        assert field("private_segment_fixed_size") == 0, f"{name} uses scratch"
        assert field("vgpr_spill_count") == 0 and field("sgpr_spill_count") == 0, name
        start = asm.index(name + ":")
        body = asm[start:asm.index(".Lfunc_end", start)]
        loads = re.findall(r"^\s+global_load_dwordx4\b.*$", body, re.M)
        assert sum(bool(re.search(r"\bnt\b", line)) for line in loads) >= 24, name
        assert "s_memrealtime" in body and "atomic" not in body, name
    assert seen == {0, 1, 2, 3}
