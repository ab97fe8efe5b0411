"""Centre selection: no LDS address is made of a register that some way to the read leaves undefined (the compiler marks those "implicit-def"): all
lanes of a wavefront look at statuses together, also those of groups that have no token to look for.  Read from the assembly; CPU only."""
from tests import asm_util as A

_NO_RESULT = ("ds_write", "global_store", "buffer_store", "scratch_store", "s_cbranch", "s_branch", "s_waitcnt", "s_nop", "s_barrier", "v_cmp", "s_cmp", "ds_add", "global_atomic")
_LOADS = ("global_load", "buffer_load", "flat_load", "scratch_load", "ds_read", "s_load", "v_readlane", "v_readfirstlane")


def _reads_at_undefined(p):
    state, work, hits = {0: frozenset()}, [0], set()
    while work:
        i = work.pop()
        bad = state[i] | p.undefined.get(i, set())
        op, _, rest = p.ins[i].partition(" ")
        args = rest.split(",")
        to = set() if op.startswith(_NO_RESULT) else A.registers(args[0])
        of = A.registers(rest if not to else ",".join(args[1:]))
        if op == "ds_read_u8" and A.registers(args[1]) & bad:
            hits.add(p.ins[i])
        bad = bad | {r for r in to if r[0] == "v"} if of & bad and not op.startswith(_LOADS) else bad - to
        for j in p.after[i]:
            if j not in state or not bad <= state[j]:
                state[j] = state.get(j, frozenset()) | bad
                work.append(j)
    return hits


def test_statuses_are_read_at_defined_positions():
    found = [(name, A.Program(body)) for name, body in A.kernels("pact_centres.hip") if "centres_kernel" in name]
    assert len(found) == 2                                          # bf16 and fp32 keys
    for name, p in found:
        assert any(t.startswith("ds_read_u8") for t in p.ins), name
        assert not _reads_at_undefined(p), name
