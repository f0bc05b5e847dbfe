"""The kernels whose matrix products are inline assembly, built with the library's
own flags, use no product's result before it is there (see asm_listing.py)."""
import pytest

from tests.asm_listing import BF16, F64, functions, listing, product_hazards

# source, product, register file of its accumulators, kernels that hold such products
CASES = [("fwd_f32.hip", F64, "v", 2), ("bwd_f32.hip", F64, "v", 4), ("bwd_dkdv.hip", BF16, "a", 8)]


@pytest.mark.parametrize("src,product,file,n", CASES, ids=[c[0] for c in CASES])
def test_products_are_waited_for(src, product, file, n):
    text = listing(src)
    if text is None:
        pytest.skip("hipcc not available")
    mine = lambda body: any(op == product and ops[0].startswith(file) for _, _, op, ops in body)  # noqa: E731
    kernels = {name: body for name, body in functions(text).items() if mine(body)}
    assert len(kernels) == n, sorted(kernels)
    bad = {name: product_hazards(body, product, file) for name, body in kernels.items()}
    assert not any(bad.values()), {name: h for name, h in bad.items() if h}


P0 = f"{F64} v[0:7], v[10:11], v[12:13], v[0:7]"
SNIPPETS = [  # (body, wait states at the early uses)
    ([P0, "s_nop 15", "s_nop 2", "v_mov_b32 v20, v7"], []),
    ([P0, "s_nop 15", "s_nop 1", "v_mov_b32 v20, v7"], [18]),
    ([P0, P0, f"{F64} v[30:37], v[10:11], v[12:13], v[30:37]", "s_nop 7", "scratch_store_dwordx2 off, v[36:37], s32"],
     [8]),
    ([P0, f"{F64} v[30:37], v[6:7], v[12:13], v[30:37]"], [0]),
    ([P0, "s_cbranch_scc1 .LBB0_2", "s_nop 15", "s_nop 7", ".LBB0_2:", "v_add_f64 v[40:41], v[0:1], v[42:43]"], [1]),
    ([".LBB0_1:", "v_mov_b64_e32 v[20:21], v[2:3]", "s_nop 7", P0, "s_nop 4", "s_branch .LBB0_1"], [6]),
]


@pytest.mark.parametrize("body,early", SNIPPETS, ids=range(len(SNIPPETS)))
def test_the_reader_counts_wait_states(body, early):
    text = "_Zkernel:\n" + "\n".join(body) + "\ns_endpgm\n.size _Zkernel\n"
    assert [h[2] for h in product_hazards(functions(text)["_Zkernel"])] == early
