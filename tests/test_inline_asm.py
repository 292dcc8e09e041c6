"""Inline assembly in the kernel sources.  The compiler keeps the distances that the hardware asks for (a vector instruction
behind the matrix instruction whose result it reads, for one) between its own instructions; it does not look into assembly
text.  So the only instructions written that way are the loads from global memory straight into LDS, whose operands are
addresses; every other block is empty and only pins a value to its place."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2506_15545_amd", "csrc")
LDS_LOAD = re.compile(r"s_mov_b32 m0, %\d; s_nop \d; global_load_lds_dwordx4 %0, (off|%1)")


def test_inline_assembly_holds_nothing_but_loads_into_lds():
    texts = []
    for path in sorted(glob.glob(os.path.join(CSRC, "*.h*p"))):
        for m in re.finditer(r'\basm\s+volatile\s*\(\s*"([^"]*)"', re.sub(r"//[^\n]*", "", open(path).read())):
            texts.append((os.path.basename(path), m.group(1).replace("\\n\\t", "; ")))
    assert sum(bool(t) for _, t in texts) == 2    # the two forms of the load
    for name, text in texts:
        assert not text or LDS_LOAD.fullmatch(text), f"{name}: {text}"
