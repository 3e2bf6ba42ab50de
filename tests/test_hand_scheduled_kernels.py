"""The kernels of csrc/sem.hip whose products and accumulator loads are inline assembly, as the compiler at hand builds them (no GPU).

The compiler neither waits for those loads nor keeps the distances that the products need: it only does not get in their way as long as
the accumulators stay in their registers and nothing is written into an operand just before its product.  The listing is walked along all its
branches for that."""
import os
import re
import subprocess

import pytest

from paper_2602_21597_amd import build

VALU_TO_PRODUCT = 2       # instructions between a vector instruction's result and a product that reads it
PRODUCT_TO_READ = 18      # ... between a product (16x16x32) and a store or copy of its result


def _regs(operand):
    m = re.fullmatch(r"([av])(\d+)|([av])\[(\d+):(\d+)\]", operand)
    if not m:
        return set()
    if m[1]:
        return {(m[1], int(m[2]))}
    return {(m[3], i) for i in range(int(m[4]), int(m[5]) + 1)}


def _blocks(body):
    """label -> (instructions as (name, operands), labels that may follow)"""
    blocks, order, label = {}, [], "start"
    cur = blocks.setdefault(label, [])
    order.append(label)
    for line in body.splitlines():
        line = line.split(";")[0].strip()
        m = re.match(r"(\.LBB\w+):", line)
        if m:
            label = m[1]
            cur = blocks.setdefault(label, [])
            order.append(label)
            continue
        if not line or line.startswith((".", "#")):
            continue
        name, _, rest = line.partition(" ")
        cur.append((name, [x.strip().split()[0] for x in rest.split(",") if x.strip()]))
    out = {}
    for i, label in enumerate(order):
        after = [ops[0] for name, ops in blocks[label] if "branch" in name]
        last = blocks[label][-1][0] if blocks[label] else ""
        if last not in ("s_branch", "s_endpgm") and i + 1 < len(order):
            after.append(order[i + 1])
        out[label] = (blocks[label], after)
    return out


def findings(body):
    """What is wrong in a kernel's listing."""
    blocks = _blocks(body)
    found = set()

    def walk(label, loading, written, product):
        """Registers that loads are on their way to; instructions still to pass after a vector write, after a product."""
        loading, written, product = set(loading), dict(written), dict(product)
        for name, ops in blocks[label][0]:
            regs = [_regs(x) for x in ops]
            acc = {r for x in regs for r in x if r[0] == "a"}
            passed = 1
            if name == "s_nop":
                passed = int(ops[0], 0) + 1
            if name == "s_waitcnt" and "vmcnt(0)" in ops:
                loading.clear()
            if name.startswith("v_mfma"):
                if regs[0] != regs[3]:
                    found.add("a product that does not accumulate in place")
                if acc & loading:
                    found.add("a product of an accumulator that is being loaded")
                if any(r in written for x in regs[1:] for r in x):
                    found.add("an operand written just before its product")
            elif acc:
                loads = name.startswith("global_load")
                if (acc & loading) - (regs[0] if loads else set()):
                    found.add("%s of an accumulator that is being loaded" % name)
                if any(r in product for r in acc):
                    found.add("%s of a result that is not there yet" % name)
                if not loads and not name.startswith(("global_store", "v_accvgpr")):
                    found.add("%s works on accumulators" % name)
            for table in (written, product):
                for r in [r for r in table if table[r] <= passed]:
                    del table[r]
                for r in table:
                    table[r] -= passed
            if name.startswith("v_mfma"):
                product.update({r: PRODUCT_TO_READ for r in regs[0]})
            elif name.startswith("v_") and regs:
                written.update({r: VALU_TO_PRODUCT for r in regs[0]})
            elif name.startswith("global_load") and "lds" not in name:
                loading |= {r for r in regs[0] if r[0] == "a"}
        return loading, written, product

    state = {"start": (set(), {}, {})}
    todo = ["start"]
    while todo:
        label = todo.pop()
        after = walk(label, *state[label])
        for nxt in blocks[label][1]:
            old = state.get(nxt)
            new = after
            if old:
                new = (old[0] | after[0],) + tuple({r: max(a.get(r, 0), b.get(r, 0)) for r in {*a, *b}} for a, b in zip(old[1:], after[1:]))
            if new != old:
                state[nxt] = new
                todo.append(nxt)
    # accumulators move only before the first product and after the last
    names = [name for label in blocks for name, _ in blocks[label][0]]
    products = [i for i, name in enumerate(names) if name.startswith("v_mfma")]
    if any(name.startswith("v_accvgpr") for name in names[products[0]:products[-1]]):
        found.add("accumulators copied between products")
    return found


@pytest.fixture(scope="module")
def listing(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("listing") / "sem.s")
    subprocess.run([build._hipcc()] + build.FLAGS + ["-x", "hip", "-S", "--cuda-device-only", os.path.join(build.CSRC, "sem.hip"), "-o", out],
                   check=True, capture_output=True)
    with open(out) as f:
        return f.read()


@pytest.mark.parametrize("kernel", ["sem_stream_kernel", "sem_wgrad_kernel"])
def test_registers_and_distances(listing, kernel):
    symbol = re.search(r"^(\w*%s\w*):" % kernel, listing, re.M)[1]
    body = re.search(r"^%s:(.*?)^\.Lfunc_end" % symbol, listing, re.M | re.S)[1]
    notes = re.search(r"- \.agpr_count:((?:(?!- \.agpr_count:).)*?)\.name: +%s\n(.*?)(?=- \.agpr_count:|\Z)" % symbol, listing, re.S)
    count = lambda key: int(re.search(r"\.%s: +(\d+)" % key, notes[2])[1])
    assert int(notes[1].split()[0]) == 208                    # 4 x 13 blocks of 4: every accumulator in a register of its own
    assert count("vgpr_count") <= 512 and count("vgpr_spill_count") == 0 and count("sgpr_spill_count") == 0
    assert count("private_segment_fixed_size") == 0
    assert findings(body) == set()
    # ... and the walk sees what it is for
    lines = body.splitlines()
    at = next(i for i, l in enumerate(lines) if "v_mfma" in l)
    operand = re.search(r"v_mfma\S+ \S+ v\[(\d+):", lines[at])[1]
    spoiled = lambda line: findings("\n".join(lines[:at] + [line] + lines[at:]))
    assert "an operand written just before its product" in spoiled("\tv_mov_b32_e32 v%s, v0" % operand)
    first = re.search(r"v_mfma\S+ (a\[\d+:\d+\])", lines[at])[1]
    assert "a product of an accumulator that is being loaded" in spoiled("\tglobal_load_dwordx4 %s, v[0:1], off" % first)
