"""The bf16 attention kernels as built: what their asynchronous loads leave behind.

The token indices of the window items are requested by inline assembly that the compiler's wait-count
bookkeeping does not see, and waited for by hand.  To the compiler the destination registers hold
their values from the request on and are free after their last use, so the source has to see to it that no
register is touched while its load is in flight.  Here the disassembly of the library built from this
tree is walked over every path of its control flow."""
import os
import re
import shutil
import subprocess

import pytest

import paper_2505_18809_amd as vorta

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
VMEM = re.compile(r"(buffer|global|flat|scratch)_(load|store|atomic)")
VREG = re.compile(r"(?<![a-z0-9_])v(?:(\d+)|\[(\d+):(\d+)\])")


def vregs(text):
    out = set()
    for one, lo, hi in VREG.findall(text):
        out.update([int(one)] if one else range(int(lo), int(hi) + 1))
    return out


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """name -> instructions [(mnemonic, operands)] and labels {name: index} of every bf16 attention kernel."""
    if not os.path.exists(OBJDUMP):
        pytest.skip("no disassembler")
    vorta.load_library()
    where = tmp_path_factory.mktemp("code")
    lib = shutil.copy(vorta.binding.LIB_PATH, where)
    subprocess.run([OBJDUMP, "--offloading", lib], check=True, capture_output=True, cwd=where)
    found = {}
    for f in sorted(os.listdir(where)):
        if not f.endswith("gfx950"):
            continue
        text = subprocess.run([OBJDUMP, "-d", "--symbolize-operands", "--no-show-raw-insn", str(where / f)], check=True,
                              capture_output=True, text=True).stdout
        name = None
        for line in text.splitlines():
            head = re.match(r"(?:[0-9a-f]+ )?<(\S+)>:", line)
            if head and not re.fullmatch(r"L\d+", head[1]):
                name = head[1] if "attn_bf16" in head[1] else None
                if name:
                    code, labels = found[name] = ([], {})
            elif head and name:
                labels[head[1]] = len(code)
            elif name and line.startswith("\t"):
                op, _, rest = line.split("//")[0].strip().partition(" ")
                code.append((op, rest.strip()))
    assert len(found) >= 9, sorted(found)
    return found


def basic_blocks(code, labels):
    """[(first, end, successors)]; an index past the code is an exit."""
    starts = {0, *labels.values()} | {i + 1 for i, (op, _) in enumerate(code) if op.startswith(("s_branch", "s_cbranch", "s_endpgm"))}
    starts = sorted(s for s in starts if s < len(code))
    at = {s: b for b, s in enumerate(starts)}
    blocks = []
    for b, s in enumerate(starts):
        e = starts[b + 1] if b + 1 < len(starts) else len(code)
        op, rest = code[e - 1]
        nxt = []
        if op.startswith(("s_branch", "s_cbranch")):
            nxt.append(at[labels[rest.strip("<>")]])
        if not op.startswith(("s_branch", "s_endpgm")) and e in at:
            nxt.append(at[e])
        assert not op.startswith(("s_setpc", "s_swappc", "s_call")), "indirect control flow"
        blocks.append((s, e, nxt))
    return blocks


def in_loop(blocks):
    """Blocks that can reach themselves."""
    reach = []
    for b in range(len(blocks)):
        seen, todo = set(), list(blocks[b][2])
        while todo:
            x = todo.pop()
            if x not in seen:
                seen.add(x)
                todo += blocks[x][2]
        reach.append(b in seen)
    return reach


def walk(code, blocks, visit, counts=lambda block: True):
    """Forward data flow.  The state maps a register to the fewest memory operations requested behind the load
    that fills it, over all paths on which that load can still be in flight (the counter retires in order, so
    after s_waitcnt vmcnt(n) a load with n or more behind it has arrived).  Loads of the blocks that `counts`
    takes are followed.  visit(index, block, state) is called with the state an instruction meets, once the
    states are stable."""
    entry = {0: {}}
    todo = [0]

    def step(i, b, state):
        op, rest = code[i]
        if op == "s_waitcnt":
            m = re.search(r"vmcnt\((\d+)\)", rest)
            if m:
                return {r: n for r, n in state.items() if n < int(m[1])}
        elif VMEM.match(op):
            state = {r: min(n + 1, 63) for r, n in state.items()}
            if counts(b) and "_load" in op and not re.search(r"\blds\b", rest) and "_lds_" not in op:
                for r in vregs(rest.split(",")[0]):
                    state[r] = 0
        return state

    while todo:
        b = todo.pop()
        state = entry[b]
        for i in range(blocks[b][0], blocks[b][1]):
            state = step(i, b, state)
        for x in blocks[b][2]:
            old = entry.get(x)
            new = dict(state) if old is None else {r: min(old.get(r, 64), state.get(r, 64)) for r in old.keys() | state.keys()}
            if new != old:
                entry[x] = new
                todo.append(x)
    for b in entry:
        state = entry[b]
        for i in range(blocks[b][0], blocks[b][1]):
            visit(i, b, state)
            state = step(i, b, state)


def test_no_register_is_touched_while_a_load_is_filling_it(kernels):
    for name, (code, labels) in kernels.items():
        touched = []

        def visit(i, b, state):
            op, rest = code[i]
            if VMEM.match(op) and "_load" in op:       # loads return in order: the later one into a register wins
                rest = rest.partition(",")[2]
            hit = vregs(rest) & state.keys()
            if hit:
                touched.append((i, code[i], sorted(hit)))

        walk(code, basic_blocks(code, labels), visit)
        assert not touched, (name, touched[:4])


def test_the_last_index_lookups_have_arrived_when_their_registers_are_free(kernels):
    """Behind the main loop of the pipelined kernel nothing reads the indices any more, so their registers are
    free for the fragments of the last product: the lookups of the loop have to be complete by then,
    whichever registers this build happens to give them."""
    checked = 0
    for name, (code, labels) in kernels.items():
        if "split" in name:        # its lookups are complete at the end of every iteration
            continue
        blocks = basic_blocks(code, labels)
        loops = in_loop(blocks)
        late = []

        def visit(i, b, state):
            if code[i][0].startswith("v_mfma") and not loops[b]:
                nonlocal checked
                checked += 1
                if state:
                    late.append((i, code[i], sorted(state)))

        walk(code, blocks, visit, counts=lambda b: loops[b])
        assert not late, (name, late[:4])
    assert checked


def test_first_scores_of_the_split_kernel_wait_for_no_later_rows(kernels):
    """The first eight matrix instructions of a stream need the queries and K(0), which the wait for all but the last eight
    loads covers; K(1) and V(0) are on their way behind them.  A wait of the compiler's own among those instructions
    (for loads that it sees, and it does not see the row loads) would take K(1) and V(0) with it."""
    for name, (code, _) in kernels.items():
        if "split" not in name:
            continue
        streams = 0
        for i, (op, rest) in enumerate(code):
            if op != "s_barrier" or ("buffer_load_dwordx4" not in [o for o, _ in code[max(0, i - 8):i]]):
                continue
            waits, products = [], 0
            for o, r in code[i:]:
                products += o.startswith("v_mfma")
                if products == 8:
                    break
                if o == "s_waitcnt" and "vmcnt" in r:
                    waits.append(r)
            if waits or not any(o == "s_waitcnt" and "vmcnt(8)" in r for o, r in code[max(0, i - 4):i]):
                pytest.fail(f"{name}: {waits}")
            streams += 1
        assert streams == 3, (name, streams)       # consecutive rows, tokens of a window, copies


def test_pipelined_iterations_begin_without_a_wait_for_fragments(kernels):
    """The fragments of an iteration's first three matrix instructions are requested ahead of the barrier of the one before and have
    arrived with it; those of the first iteration are waited for ahead of the loop.  Anything else in flight on the way into the
    loop makes the compiler wait at its head, in every iteration."""
    checked = 0
    for name, (code, labels) in kernels.items():
        if "split" in name:
            continue
        for i, (op, rest) in enumerate(code):
            head = labels.get(rest.strip("<>"), i) if op.startswith(("s_branch", "s_cbranch")) else i
            products = [k for k in range(head, i) if code[k][0].startswith("v_mfma")]
            # two iterations of 16 or 32 matrix instructions and a barrier each: the main loop, and no span of other code around it
            if len(products) not in (32, 64) or [op for op, _ in code[head:i]].count("s_barrier") != 2:
                continue
            late = [rest for op, rest in code[head:products[2]] if op == "s_waitcnt" and "lgkmcnt" in rest]
            assert not late, (name, late)
            checked += 1
    assert checked >= 8, checked


def test_window_blocks_that_outweigh_the_row_are_not_redone(kernels):
    """A block of window keys that weighs more than twice all before it has its sum taken of the rounded probabilities (v_dot2).
    Peaked scores have many such blocks: the way there from the matrix instructions of the iteration leads past the
    exponentials and the rescaled accumulators of a block that is redone."""
    checked = 0
    for name, (code, labels) in kernels.items():
        if "ILi0E" in name:          # dense and core-set items only
            continue
        blocks = basic_blocks(code, labels)
        before = {}
        for b, (_, _, nxt) in enumerate(blocks):
            for x in nxt:
                before.setdefault(x, []).append(b)
        ops = [[op for op, _ in code[s:e]] for s, e, _ in blocks]
        sums = [b for b in range(len(blocks)) if any(op.startswith("v_dot2") for op in ops[b])]
        assert sums, name
        for b in sums:
            seen, todo, found = set(), [b], False
            while todo and not found:
                for x in before.get(todo.pop(), []):
                    if any(op.startswith("v_mfma") for op in ops[x]):
                        found = True
                    elif x not in seen and not any(op.startswith(("v_exp", "v_mul_f32")) for op in ops[x]):
                        seen.add(x)
                        todo.append(x)
            assert found, (name, blocks[b])
            checked += 1
    assert checked
