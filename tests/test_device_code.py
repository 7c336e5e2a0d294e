"""What the kernels rely on and a run does not show, checked in the compiled code."""
import re

import code_objects as co


def _blocks(code):
    """Basic blocks of a kernel: [(instructions, successors)]; the first one is the entry."""
    index = {a: i for i, (a, _, _) in enumerate(code)}
    cuts = {0} | {index[t] for _, _, t in code if t is not None} | {i + 1 for i, (_, op, t) in enumerate(code) if t is not None or op == "s_endpgm"}
    cuts = sorted(c for c in cuts if c < len(code))
    number = {c: n for n, c in enumerate(cuts)}
    out = []
    for c, end in zip(cuts, cuts[1:] + [len(code)]):
        _, op, target = code[end - 1]
        follow = [] if op.startswith(("s_endpgm", "s_branch")) else [end]
        out.append(([o for _, o, _ in code[c:end]], [number[i] for i in follow + ([index[target]] if target is not None else []) if i in number]))
    return out


def _writes_under_way_at_barriers(code):
    """Barriers at which an LDS write of the wave may still be under way.  LDS operations end in order, so a wait
    for the counter to fall to n covers a write that n later LDS operations or more have followed.  State on the
    way through the code: how many have followed the youngest write that no wait has covered (None: no such
    write), the least over all ways that lead here."""
    blocks = _blocks(code)
    entry, todo, bad = {0: None}, [0], set()
    while todo:
        n = todo.pop()
        later, (ops, follow) = entry[n], blocks[n]
        for i, op in enumerate(ops):
            if op.startswith("ds_write"):
                later = 0
            elif op.startswith("ds_"):
                later = None if later is None else later + 1
            elif op.startswith("s_waitcnt"):
                m = re.search(r"lgkmcnt\((\d+)\)", op)
                if m and later is not None and int(m[1]) <= later:
                    later = None
            elif op.startswith("s_barrier") and later is not None:
                bad.add((n, i))
        for f in follow:
            known = entry.get(f, "new")
            if known == "new" or (later is not None and (known is None or later < known)):
                entry[f] = later
                todo.append(f)
    return bad


def test_lds_writes_end_before_the_barrier_that_publishes_them():
    """No wave passes a barrier with a write to LDS of its own still under way: the others read behind it."""
    seen, bad = set(), {}
    for name, code in co.instructions():
        seen.add(name.split("<")[0])
        n = len(_writes_under_way_at_barriers(code))
        if n:
            bad[name] = n
    assert {"gemm_mid", "gemm_skinny", "gemm_thin", "tree_attention_mfma", "f32_product", "tree_build_kernel"} <= seen
    assert not bad


def test_no_kernel_keeps_registers_in_memory():
    """Scratch memory means spilled registers, whose loads also come between those that the product kernels count."""
    used = dict(co.scratch_bytes())
    assert {n.split("<")[0] for n in used} >= {"gemm_mid", "gemm_skinny", "gemm_thin", "tree_attention_mfma", "f32_product"}
    assert not {n: b for n, b in used.items() if b}
