#!/usr/bin/env python3
"""Build step: check the generated code of the gemm_bf16_w4_kernel instantiations (the gfx950 .s file that
hipcc -save-temps leaves beside gemm.o).

The kernel issues its operand loads as asm and counts them itself, so the compiler does not know which
registers have a load in flight.  This follows every path through the kernel up to its epilogue - out-of-line blocks
included, wherever the compiler put them - with the queue of loads in flight (s_waitcnt vmcnt(N) retires the oldest down to N)
and reports any instruction that names a register whose load has not been waited for, any scratch access inside a main loop or with
loads in flight, any load behind a main loop and any load still in flight where the epilogue begins.

One thing is taken from the source: the wait for all loads at the end of a main loop's body is skipped exactly when the loop goes
on.  A path that skips it is not followed out of the loop, nor one that takes it back into it."""
import re, sys

def regs(tok):
    out = set()
    for m in re.finditer(r'\bv\[(\d+):(\d+)\]', tok):
        out.update(range(int(m.group(1)), int(m.group(2)) + 1))
    for m in re.finditer(r'\bv(\d+)\b', tok):
        out.add(int(m.group(1)))
    return out

# the epilogue, whose loads and stores the compiler knows, begins with wait states or, at the latest, with a store
EPILOGUE = re.compile(r's_nop 15\s*$|global_store|buffer_store|s_endpgm')
MAX_STATES = 200000

class Block:
    def __init__(self, start):
        self.start, self.lines, self.to = start, [], []      # (line number, text); successors

def blocks_of(code):
    """Basic blocks by the line they start at; None and a message where a jump leads nowhere known."""
    labels = {m.group(1): i for i, l in enumerate(code) for m in [re.match(r'^(\.LBB\w+):', l)] if m}
    starts = {0} | set(labels.values())
    for i, l in enumerate(code):
        if re.search(r'\bs_c?branch|\bs_setpc|\bs_endpgm', l):
            starts.add(i + 1)
    starts = sorted(s for s in starts if s < len(code))
    out = {}
    for s, e in zip(starts, starts[1:] + [len(code)]):
        b = out[s] = Block(s)
        for i in range(s, e):
            l = code[i].strip()
            if not l or l.startswith(('.', ';')) or l.endswith(':'):
                continue
            b.lines.append((i, l))
            if 's_endpgm' in l:
                break
            m = re.match(r's_(c?)branch\S*\s+(\S+)', l)
            if m:
                if m.group(2) not in labels:
                    return None, f"line {i}: jump to unknown {m.group(2)}"
                b.to = [labels[m.group(2)]] + ([e] if m.group(1) and e in starts else [])
                break
            if l.startswith('s_setpc'):
                # a far jump: the target stands in the addition to the program counter in front of it
                t = [m.group(1) for _, x in b.lines[-4:] for m in [re.match(r's_add_u32\s.*\((\.LBB\w+)-', x)] if m]
                if not t or t[-1] not in labels:
                    return None, f"line {i}: {l} without a known target"
                b.to = [labels[t[-1]]]
                break
        else:
            if e in starts:
                b.to = [e]
    return out, None

def components(blocks):
    """Strongly connected components (block start -> component number), iteratively."""
    num, low, comp, stack, on = {}, {}, {}, [], set()
    for root in blocks:
        if root in num:
            continue
        work = [(root, iter(blocks[root].to))]
        num[root] = low[root] = len(num)
        stack.append(root); on.add(root)
        while work:
            v, it = work[-1]
            for w in it:
                if w not in num:
                    num[w] = low[w] = len(num)
                    stack.append(w); on.add(w)
                    work.append((w, iter(blocks[w].to)))
                    break
                if w in on:
                    low[v] = min(low[v], num[w])
            else:
                work.pop()
                if work:
                    low[work[-1][0]] = min(low[work[-1][0]], low[v])
                if low[v] == num[v]:
                    while True:
                        w = stack.pop(); on.discard(w)
                        comp[w] = v
                        if w == v:
                            break
    return comp

def is_load(l):
    return 'buffer_load_dwordx4' in l

def check(name, lines):
    code = [l.split(';')[0].rstrip() for l in lines]
    n_loops = 2 if 'ILi0ELi0E' in name else 1      # the NT kernel has a second loop for two passes
    n_bar = sum('s_barrier' in l for l in code)
    if n_bar != 5 * n_loops:
        return False, f"{name}: expected 5 barriers (prologue, two loop phases, two tail phases) for each of {n_loops} loops, found {n_bar}"
    blocks, err = blocks_of(code)
    if err:
        return False, f"{name}: {err}"
    comp = components(blocks)
    cyclic = {comp[s] for s, b in blocks.items() for t in b.to if comp[t] == comp[s]}
    loops = {}
    for s, b in blocks.items():
        if comp[s] in cyclic:
            loops.setdefault(comp[s], []).append(b)
    loops = {c: bs for c, bs in loops.items() if any(is_load(l) for b in bs for _, l in b.lines)}
    bad = []
    if len(loops) != n_loops:
        return False, f"{name}: expected {n_loops} main loops, found {len(loops)}"
    drains = {}      # loop -> block with its wait for all loads
    for c, bs in loops.items():
        if sum('s_barrier' in l for b in bs for _, l in b.lines) != 2:
            bad.append((0, "a main loop without its two barriers"))
        drains[c] = [b.start for b in bs if any(re.search(r's_waitcnt vmcnt\(0\)', l) for _, l in b.lines)]
        if not drains[c]:
            bad.append((0, "no vmcnt(0) drain in the loop body"))
    # code behind a main loop: what its exits reach
    behind, todo = set(), [t for c, bs in loops.items() for b in bs for t in b.to if comp[t] != c]
    while todo:
        s = todo.pop()
        if s not in behind:
            behind.add(s)
            todo += blocks[s].to

    stat = dict(maxq=0, waits=set(), states=0)
    def run(b, queue):
        """One block: the queue behind it, or None where the epilogue begins."""
        q = list(queue)
        in_loop = comp[b.start] in loops
        for i, l in b.lines:
            if EPILOGUE.search(l):
                if q:
                    bad.append((i, "loads in flight at the epilogue"))
                return None
            if l.startswith('s_waitcnt'):
                m = re.search(r'vmcnt\((\d+)\)', l)
                if m:
                    n = int(m.group(1))
                    if n:
                        stat['waits'].add(i)
                    q = q[len(q) - n:] if len(q) > n else q
                    if n == 0:
                        q = []
                continue
            pending = set().union(*q) if q else set()
            if ('scratch_' in l and (in_loop or q)) or (regs(l) & pending):
                bad.append((i, l))
            if is_load(l):
                if b.start in behind:
                    bad.append((i, "loads issued behind the loop: " + l))
                q.append(frozenset(regs(l.split(',')[0])))
                stat['maxq'] = max(stat['maxq'], len(q))
        return tuple(q)

    seen = set()
    def explore(first):
        todo = [(first, (), None)]
        while todo:
            s, queue, went = state = todo.pop()
            if state in seen:
                continue
            seen.add(state)
            if len(seen) > MAX_STATES or len(bad) > 200:
                bad.append((0, "too many paths")) if len(seen) > MAX_STATES else None
                return
            b = blocks[s]
            out = run(b, queue)
            if out is None:
                continue
            c = comp[s]
            if s in drains.get(c, ()):
                went = 'out'
            leaves = [t for t in b.to if comp[t] != c]
            for t in b.to:
                skips = c in loops and len(b.to) == 2 and t not in drains[c] and any(d in drains[c] and t in blocks[d].to for d in b.to)
                w = 'on' if skips else went
                if c in loops and leaves and len(b.to) == 2 and w:      # the loop's own test
                    if (t in leaves) != (w == 'out'):
                        continue
                    w = None
                todo.append((t, out, w if comp[t] == c else None))
    explore(min(blocks))
    # code that neither a path nor the epilogue reaches is walked with nothing in flight, as code behind a loop
    known, todo = set(), [s for s, _, _ in seen]
    while todo:
        s = todo.pop()
        if s not in known:
            known.add(s)
            todo += blocks[s].to
    for s in sorted(set(blocks) - known):
        behind.add(s)
        explore(s)
    if stat['maxq'] > 48:
        bad.append((0, "more than 48 loads in flight"))
    msg = f"{name}: {n_loops} main loop(s) of {', '.join(str(sum(len(b.lines) for b in bs)) for bs in loops.values())} instructions, {len(seen)} states, at most {stat['maxq']} loads in flight, {len(stat['waits'])} counted waits"
    if bad:
        return False, msg + "\n  VIOLATIONS:\n" + "\n".join(f"    line {i}: {l}" for i, l in sorted(set(bad))[:20])
    return True, msg + "  OK"

def main(path):
    txt = open(path).read().split('\n')
    starts = [(i, m.group(1)) for i, l in enumerate(txt) for m in [re.match(r'^(_ZN\S*gemm_bf16_w4_kernel\S*):', l)] if m]
    rc = 0 if starts else 1
    for i, nm in starts:
        j = next(k for k in range(i, len(txt)) if txt[k].startswith('.Lfunc_end'))
        ok, r = check(nm[-40:], txt[i:j])
        print(r)
        rc |= 0 if ok else 1
    if not starts:
        print("no w4 kernels in", path)
    return rc

if __name__ == '__main__':
    sys.exit(main(sys.argv[1]))
