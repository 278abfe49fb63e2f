"""The attention's transfer loop as compiled: the waits on global memory in it are the hand-written ones. The compiler
does not see the K/V transfers; one wait of its own on a load from before the loop would drain them at every tile."""
import os
import re
import subprocess

import pytest

from paper_2608_04962_amd import build as b


@pytest.fixture(scope="module")
def listing(tmp_path_factory):
    out = os.path.join(tmp_path_factory.mktemp("isa"), "k_attn.s")
    cmd = [b.hipcc(), *b.HIPCC_FLAGS, "-I", b.INCLUDE, "-I", b.CSRC, "-S", "--cuda-device-only",
           os.path.join(b.CSRC, "k_attn.hip"), "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    with open(out) as f:
        return f.read().split("\n")


def _transfer_loop(lines):
    """(line, in inline asm) from the first to the last block of the loop that both meets the block and issues
    transfers. Blocks name the header of their innermost loop in the compiler's comments."""
    spans, header, label, asm, marked = {}, None, None, False, []
    for n, ln in enumerate(lines):
        m = re.match(r"(?:\.L(BB\d+_\d+):|; %bb\.\d+:)(.*)", ln)
        if m:
            label = m.group(1) or label
            h = re.search(r"Header=(BB\d+_\d+)", m.group(2))
            header = h.group(1) if h else label if "Loop Header" in m.group(2) else None
        elif "Loop Header" in ln and ln.lstrip().startswith(";"):
            header = label
        asm = "#ASMSTART" in ln or (asm and "#ASMEND" not in ln)
        marked.append((ln.strip(), asm))
        if header:
            s = spans.setdefault(header, dict(first=n, last=n, sync=False, issue=False))
            s["last"] = n
            s["sync"] |= asm and "s_barrier" in ln
            s["issue"] |= asm and "global_load_lds" in ln
    found = [s for s in spans.values() if s["sync"] and s["issue"]]
    assert len(found) == 1, spans
    return marked[found[0]["first"]:found[0]["last"] + 1]


@pytest.mark.parametrize("D", [64, 128])
def test_no_compiler_wait_in_the_transfer_loop(listing, D):
    i = next(n for n, ln in enumerate(listing) if re.match(rf"_ZN2sr15k_tree_attn_dmaILi{D}E\S*:", ln))
    j = next(n for n in range(i, len(listing)) if listing[n].startswith(".Lfunc_end"))
    body = _transfer_loop(listing[i:j])
    assert sum("global_load_lds" in t for t, _ in body) >= 2 * 64 * D * 2 // 1024   # a tile's transfers
    own = [t for t, asm in body if not asm and ("vmcnt" in t or t.startswith(("scratch_", "global_", "flat_", "buffer_")))]
    assert not own, own
