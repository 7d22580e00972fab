"""Stores of more than 8 bytes written in assembly carry the wait states that the hardware asks for and the compiler cannot add: on gfx950
the two vector instructions after such a store must not write its data registers."""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_20524_amd", "csrc")


def test_wide_stores_in_assembly_are_followed_by_two_wait_states():
    stores = []
    for name in sorted(os.listdir(CSRC)):
        if not name.endswith((".hip", ".h")):
            continue
        with open(os.path.join(CSRC, name)) as f:
            stores += [(name, m.group(0)) for m in re.finditer(r'(?:global|buffer|flat)_store_(?:dwordx[34]|b96|b128)[^"]*"', f.read())]
    assert stores
    for name, text in stores:
        nop = re.search(r"\\n\\ts_nop (\d+)", text)
        assert nop and int(nop.group(1)) >= 1, (name, text)
