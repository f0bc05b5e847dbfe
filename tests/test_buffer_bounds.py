"""Rows past the end of a range read as zeros because the buffer resource ends
with the range; the bounds check takes the vector offset only, so no access may
put part of the row's address into the scalar offset (see asm_listing.py).  The
sources here load through builtins with a choice of both."""
import pytest

from tests.asm_listing import functions, listing, scalar_offset_accesses

@pytest.mark.parametrize("src", ["fwd_f32.hip", "bwd_f32.hip", "merge.hip"])
def test_no_row_address_in_a_scalar_offset(src):
    text = listing(src)
    if text is None:
        pytest.skip("hipcc not available")
    found = {n: scalar_offset_accesses(b) for n, b in functions(text).items()}
    assert sum(n for n, _ in found.values()) > 0
    assert not any(lines for _, lines in found.values()), {n: x[1] for n, x in found.items() if x[1]}
