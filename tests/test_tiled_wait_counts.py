"""The written-out wait counts of the matrix-core expert kernel, checked against the code the
compiler produced.

The kernel copies token tiles global -> LDS with instructions the compiler does not track and
orders them with ``s_waitcnt vmcnt(N)`` written next to every barrier.  Vector-memory
instructions of a wavefront complete in issue order, so the wait guarantees "every copy but the
most recent K has landed" exactly when at least N vector-memory instructions were issued after the
last copy before those K.  K is the copies of the steps that may still be on their way: a step of a
tile of NJ 32-row sub-tiles issues NJ, and floor(kNP / NJ) steps are (kNP: copies of a full tile's
step).  The kernel writes K into a comment beside each wait.  Part of the N are weight loads
whose position the compiler chooses, so the property is verified here, on the assembly text the
device object is assembled from, at every such wait of every instantiation and along every path
that reaches it.  No GPU needed.
"""
import os
import re
import subprocess

import pytest

from paper_2505_06481_amd import build as mbuild

SRC = os.path.join(mbuild.CSRC, "ffn_tiled.hip")

VM_PREFIXES = ("global_load", "global_store", "global_atomic", "buffer_load", "buffer_store", "buffer_atomic",
               "flat_load", "flat_store", "flat_atomic", "scratch_load", "scratch_store")
COPY = "global_load_lds_dwordx4"


def device_assembly():
    """Assembly of ffn_tiled.hip for gfx950: the file the in-tree build left behind if it is
    newer than the source, otherwise a fresh compile with the same flags."""
    deps = [SRC] + mbuild._headers()
    if os.path.exists(mbuild.TILED_ASM) and os.path.getmtime(mbuild.TILED_ASM) >= max(map(os.path.getmtime, deps)):
        return open(mbuild.TILED_ASM).read()
    os.makedirs(mbuild.OBJ_DIR, exist_ok=True)
    out = os.path.join(mbuild.OBJ_DIR, "ffn_tiled_check.s")
    subprocess.run([mbuild.HIPCC] + mbuild.FLAGS + ["--cuda-device-only", "-S", SRC, "-o", out], check=True,
                   stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    return open(out).read()


class Func:
    """Basic blocks of one function: instruction lists, successor and predecessor edges."""

    def __init__(self, name, lines):
        self.name = name
        self.blocks = []     # list of instruction lists
        label_at = {}        # label -> block index
        cur = []
        self.blocks.append(cur)
        for ln in lines:
            # a wait keeps the number in its comment, as a second operand
            m = re.search(r"; copies in flight: (\d+)", ln)
            ln = ln.split(";")[0].rstrip() + (f", {m.group(1)}" if m else "")
            if not ln.strip():
                continue
            m = re.match(r"^(\.LBB\w+):", ln)
            if m:
                if cur:
                    cur = []
                    self.blocks.append(cur)
                label_at[m.group(1)] = len(self.blocks) - 1
                continue
            if not ln.startswith("\t") or ln.lstrip().startswith("."):
                continue
            ins = ln.strip()
            cur.append(ins)
            if ins.startswith(("s_branch", "s_cbranch", "s_endpgm")):
                cur = []
                self.blocks.append(cur)
        self.succ = [[] for _ in self.blocks]
        for b, ins_list in enumerate(self.blocks):
            last = ins_list[-1] if ins_list else ""
            if last.startswith("s_endpgm"):
                continue
            if last.startswith(("s_branch", "s_cbranch")):
                self.succ[b].append(label_at[last.split()[-1]])
                if last.startswith("s_branch"):
                    continue
            if b + 1 < len(self.blocks):
                self.succ[b].append(b + 1)
        self.pred = [[] for _ in self.blocks]
        for b, ss in enumerate(self.succ):
            for t in ss:
                self.pred[t].append(b)


def functions(text, prefix):
    out = []
    for m in re.finditer(r"^(%s\w*):.*?^\.Lfunc_end\d+:" % re.escape(prefix), text, re.S | re.M):
        out.append(Func(m.group(1), m.group(0).splitlines()[1:]))
    return out


def wait_sites(fn):
    """(block, index, N, K) of every written-out "s_waitcnt vmcnt(N) ; copies in flight: K ; s_barrier"."""
    sites = []
    for b, ins_list in enumerate(fn.blocks):
        for i, ins in enumerate(ins_list[:-1]):
            if re.match(r"s_waitcnt\b.*\bvmcnt\(", ins) and ins_list[i + 1].startswith("s_barrier"):
                m = re.match(r"s_waitcnt\s+vmcnt\((\d+)\)\s*, (\d+)$", ins)
                assert m, f"{fn.name}: a wait in front of a barrier without its number of copies: {ins}"
                sites.append((b, i, int(m.group(1)), int(m.group(2))))
    return sites


def min_issued_since_older_copies(fn, block, index, k):
    """Over every path that reaches the wait: the number of vector-memory instructions issued
    after the last copy that must have landed (the (k+1)-th copy, walking backwards).  Returns the
    minimum, or None if some path reaches the function entry first."""
    best = [None]
    seen = set()
    stack = [(block, index, 0, 0)]   # block, instructions of it still to scan, copies seen, vm ops seen
    while stack:
        b, n, copies, vm = stack.pop()
        done = False
        for ins in reversed(fn.blocks[b][:n]):
            if ins.startswith(VM_PREFIXES):
                if ins.startswith(COPY):
                    copies += 1
                    if copies == k + 1:
                        best[0] = vm if best[0] is None else min(best[0], vm)
                        done = True
                        break
                vm += 1
        if done:
            continue
        if not fn.pred[b]:
            return None
        for p in fn.pred[b]:
            key = (p, copies, vm)
            if key not in seen:
                seen.add(key)
                stack.append((p, len(fn.blocks[p]), copies, vm))
    return best[0]


def check_function(fn):
    """List of (N, K, issued) for every written-out wait; raises on a violated one."""
    res = []
    for b, i, n, k in wait_sites(fn):
        issued = min_issued_since_older_copies(fn, b, i, k)
        assert issued is not None, f"{fn.name}: a path reaches the wait before {k + 1} copies were issued"
        assert issued >= n, (f"{fn.name}: s_waitcnt vmcnt({n}) is preceded by only {issued} vector-memory "
                             f"instructions since the copies that must have landed: one could still be in flight")
        res.append((n, k, issued))
    return res


def variants(name):
    """(NJ, K, number of waits) of every height a tile of this instantiation can have."""
    bm, nb = (int(x) for x in re.search(r"ILi\d+ELi(\d+)ELi(\d+)EE", name).groups())
    knp = bm * 8 // 256                                   # copies per wavefront and step of a full tile
    steps_per_trip = 4 if bm == 256 or nb == 1 else 2
    # one wait in the prologue and one per unrolled step of the main loop
    return [(nj, knp // nj * nj, 1 + steps_per_trip) for nj in range(1, bm // 32 + 1)]


def test_checker_flags_a_short_window():
    """The checker itself: a hand-written stream in which a weight load has been moved from behind
    the copies to in front of them must be refused, the original accepted."""
    def stream(loads_after):
        body = ["\tglobal_load_lds_dwordx4 v1, s[0:1]"] * 2                     # older group
        body += ["\tglobal_load_dwordx4 v[2:5], v[6:7], off"] * (3 - loads_after)
        body += ["\tglobal_load_lds_dwordx4 v1, s[0:1]"] * 2                    # older group
        body += ["\tglobal_load_dwordx4 v[2:5], v[6:7], off"] * loads_after
        body += ["\tglobal_load_lds_dwordx4 v1, s[0:1]"] * 2                    # most recent group
        body += ["\ts_waitcnt vmcnt(5) ; copies in flight: 2", "\ts_barrier", "\ts_endpgm"]
        return Func("f", body)
    assert check_function(stream(3)) == [(5, 2, 5)]
    with pytest.raises(AssertionError):
        check_function(stream(2))
    # a loop: the window wraps around the back edge
    loop = Func("g", ["\tglobal_load_lds_dwordx4 v1, s[0:1]", ".LBB9_1:",
                      "\tglobal_load_dwordx4 v[2:5], v[6:7], off", "\ts_waitcnt vmcnt(2) ; copies in flight: 1", "\ts_barrier",
                      "\tglobal_load_lds_dwordx4 v1, s[0:1]", "\ts_cbranch_scc1 .LBB9_1", "\ts_endpgm"])
    with pytest.raises(AssertionError):     # first trip: only one copy precedes the wait
        check_function(loop)
    # a wait that does not say what it leaves in flight
    with pytest.raises(AssertionError):
        check_function(Func("h", ["\tglobal_load_lds_dwordx4 v1, s[0:1]", "\ts_waitcnt vmcnt(0)", "\ts_barrier"]))


def test_every_written_out_wait_of_the_tiled_kernel_is_covered():
    text = device_assembly()
    fns = functions(text, "_ZN4mmoe12tiled_kernel")
    # 4 products (three activations, down) x 2 tile heights, and the three products without a gate
    # once more with one weight block per wavefront (128-row tiles only)
    assert len(fns) == 14, [f.name for f in fns]
    for fn in fns:
        res = check_function(fn)
        want = sorted(k for _, k, waits in variants(fn.name) for _ in range(waits))
        assert sorted(k for _, k, _ in res) == want, fn.name
        print(f"{fn.name}: {len(res)} waits, smallest margin {min(i - n for n, _, i in res)}")


def test_waits_of_the_kernel_for_slots_of_one_tile():
    """The same main loops, each twice: weights through the caches and past them."""
    fns = functions(device_assembly(), "_ZN4mmoe17tiled_lone_kernel")
    assert len(fns) == 5, [f.name for f in fns]
    for fn in fns:
        mode = re.search(r"kernelILi(\d)E", fn.name).group(1)
        res = check_function(fn)
        want = sorted(k for _, k, waits in variants(f"_ZN4mmoe12tiled_kernelILi{mode}ELi256ELi2EE") for _ in range(2 * waits))
        assert sorted(k for _, k, _ in res) == want, fn.name


def test_waits_of_the_128_row_kernel_for_slots_of_one_tile():
    """As above: five products with two weight blocks per wavefront, the four without a gate with one too."""
    fns = functions(device_assembly(), "_ZN4mmoe23tiled_lone_small_kernel")
    assert len(fns) == 9, [f.name for f in fns]
    for fn in fns:
        mode, nb = re.search(r"kernelILi(\d)ELi(\d)E", fn.name).groups()
        res = check_function(fn)
        want = sorted(k for _, k, waits in variants(f"_ZN4mmoe12tiled_kernelILi{mode}ELi128ELi{nb}EE") for _ in range(2 * waits))
        assert sorted(k for _, k, _ in res) == want, fn.name


def test_waits_of_the_256_row_kernel_of_128_features():
    """The four products without a gate, each as for batches of many rows and (weights past the caches too) for slots of one tile."""
    fns = functions(device_assembly(), "_ZN4mmoe19tiled_narrow_kernel")
    assert len(fns) == 8, [f.name for f in fns]
    for fn in fns:
        mode, lone = re.search(r"kernelILi(\d)ELb([01])E", fn.name).groups()
        res = check_function(fn)
        times = 1 + int(lone)
        want = sorted(k for _, k, waits in variants(f"_ZN4mmoe12tiled_kernelILi{mode}ELi256ELi1EE") for _ in range(times * waits))
        assert sorted(k for _, k, _ in res) == want, fn.name


def test_loads_moved_across_a_wait_are_flagged():
    """A mistake planted in the assembly text: the waits with one number of copies in flight (tiles of 3, 5, 6 and 7
    sub-tiles have their own) leave three more instructions outstanding than the kernel asks for, as if three loads had
    been moved behind them.  Every kernel must be refused for each of its numbers."""
    text = device_assembly()
    for name in sorted({fn.name for fn in functions(text, "_ZN4mmoe12tiled_kernel")}):
        body = re.search(r"^%s:.*?^\.Lfunc_end\d+:" % re.escape(name), text, re.S | re.M).group(0).splitlines()[1:]
        for k in sorted({k for _, k, _ in variants(name)}):
            pat = r"s_waitcnt vmcnt\((\d+)\) ; copies in flight: %d$" % k
            moved = [re.sub(pat, lambda m: f"s_waitcnt vmcnt({int(m.group(1)) + 3}) ; copies in flight: {k}", ln.rstrip())
                     for ln in body]
            assert moved != [ln.rstrip() for ln in body]
            with pytest.raises(AssertionError, match="could still be in flight"):
                check_function(Func(name, moved))
