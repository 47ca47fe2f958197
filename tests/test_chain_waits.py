"""The bf16 chains wait for their weight tiles by count: a wait names how many of the wavefront's youngest memory
instructions may still be on their way, and among those it counts loads and stores of rows beside the tiles.  If the compiler
dropped one of these, a tile might be read before it has arrived, and no test of results would reliably show it.  So the
built kernels are read: before each barrier of the ring, on every way through the code, the tiles that the sets up to the
next barrier read have to lie behind the wait.

A tile is LPT instructions per wavefront (8 KB, 1 KB each, over the wavefronts of a block).  Set i of eight products is
preceded by the loads of tile i + 6; the start waits for tiles 0 and 1, the barrier of set i for those up to i + 2."""
import os
import re
import subprocess
from collections import defaultdict
from heapq import heappop, heappush

import pytest

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2601_09026_amd", "libmgrit_hip.so")
OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
LEAD, G = 6, 2
LEAST = {"chain_head_kernel": (2, 8), "chain_adjoint_head_kernel": (1, 7), "chain_tail_kernel": (3, 5),
         "chain_adjoint_tail_kernel": (2, 5)}          # barriers of the 64 and the 128 wide forms; more where code is doubled
MEM = re.compile(r"(buffer|global|flat|scratch)_(load|store|atomic)")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """name -> [(address, instruction)] of the kernels of chain.hip"""
    if not os.path.exists(LIB):
        import __graft_entry__
        __graft_entry__.build()
    d = tmp_path_factory.mktemp("objects")
    lib = d / "lib.so"
    lib.symlink_to(LIB)
    subprocess.check_call([OBJDUMP, "--offloading", str(lib)], stdout=subprocess.DEVNULL, cwd=d)
    out = {}
    for f in sorted(os.listdir(d)):
        if "gfx950" not in f or b"chain_tail_kernel" not in (d / f).read_bytes():
            continue
        code = None
        for line in subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(d / f)], check=True, text=True,
                                   stdout=subprocess.PIPE).stdout.splitlines():
            m = re.match(r"[0-9a-f]+ <_ZN2mg12_GLOBAL__N_1\d+(chain_\w+_kernel)I((?:Li\d+E)+)E", line)
            if m:
                code = out.setdefault((m[1], tuple(map(int, re.findall(r"Li(\d+)E", m[2])))), [])
            m = re.match(r"\t(.*?)\s*// ([0-9A-F]+):(.*)", line)
            if m and code is not None:
                target = re.search(r"\+0x([0-9a-f]+)>", m[3])
                code.append((int(m[2], 16), m[1].strip(), int(target[1], 16) if target else 0))
    return out


class Code:
    """The memory instructions and ring barriers of a kernel and the ways between them, straight runs without any left out."""

    def __init__(self, ins):
        base, index = ins[0][0], {a: i for i, (a, _, _) in enumerate(ins)}
        self.kind, self.before, self.syncs = {}, defaultdict(list), []
        nxt = defaultdict(list)
        for i, (_, s, target) in enumerate(ins):
            if MEM.match(s):
                self.kind[i] = "tile" if s.endswith(" lds") else "other"
            if s.startswith("s_barrier"):
                j = i - 1
                while j not in self.kind and not (w := re.fullmatch(r"s_waitcnt vmcnt\((\d+)\)", ins[j][1])):
                    j -= 1
                self.syncs.append((j, int(w[1])))
            if s.startswith(("s_branch", "s_cbranch")):
                nxt[i].append(index[base + target])
            if not s.startswith(("s_branch", "s_endpgm", "s_setpc")) and i + 1 < len(ins):
                nxt[i].append(i + 1)
        for i, to in nxt.items():
            for j in to:
                self.before[j].append(i)

    def behind(self, sync, tiles):
        """The fewest memory instructions between the (tiles + 1)-th youngest tile instruction before `sync` and the sync,
        over all ways that lead there."""
        seen, heap = set(), [(0, 0, sync)]
        while heap:
            dist, passed, i = heappop(heap)
            if (passed, i) in seen:
                continue
            seen.add((passed, i))
            for j in self.before[i]:
                k = self.kind.get(j)
                if k == "tile" and passed == tiles:
                    return dist
                heappush(heap, (dist + (k is not None), passed + (k == "tile"), j))
        return None


def check(name, par, ins):
    """Every wait of the ring in one kernel; returns how many barriers there are."""
    c, d, lpt = Code(ins), par[0], 8 // par[1]
    head = name in ("chain_head_kernel", "chain_adjoint_head_kernel")
    total = 12 if d == 128 else 3                      # tiles of a head, which is one run of code
    for n, (sync, count) in enumerate(c.syncs):
        if count == 0:
            continue                                   # everything
        if head:
            s = 2 * n - (3 if name == "chain_head_kernel" else 1)                 # the set that it lies in; -1 the start
            if s < -1:
                continue                               # the rows and vectors alone, tested below
            tiles = min(max(s, 0) + LEAD, total) - min(s + 1 + G, total)
        else:
            tiles = LEAD - G if n == 0 else LEAD - G - 1
        got = c.behind(sync, tiles * lpt)
        assert got is not None and got >= count, \
            f"{name}{par}: wait {n} leaves {count} instructions open, {got} of them certainly behind the tiles it is for"
    return len(c.syncs)


def test_tiles_have_arrived_when_they_are_read(kernels):
    assert len(kernels) == 24
    for (name, par), ins in kernels.items():
        assert check(name, par, ins) >= LEAST[name][par[0] // 128], (name, par)


def test_rows_of_a_head_have_arrived(kernels):
    """The first wait of a head leaves the tiles alone open: rows and vectors were asked for before any."""
    for (name, par), ins in kernels.items():
        if name != "chain_head_kernel":
            continue
        c = Code(ins)
        sync, count = c.syncs[0]
        assert count == min(LEAD, 12 if par[0] == 128 else 3) * (8 // par[1])
        assert all(k == "tile" for i, k in sorted((i, k) for i, k in c.kind.items() if i < sync)[-count:])


def test_a_dropped_instruction_is_found(kernels):
    """The reading itself: without one of the row loads or stores that a wait counts it must fail."""
    for name, par, pick in (("chain_adjoint_tail_kernel", (128, 4), "buffer_load"), ("chain_adjoint_tail_kernel", (64, 2), "buffer_load"),
                            ("chain_tail_kernel", (128, 4, 2), "buffer_store"), ("chain_tail_kernel", (128, 4, 0), "global_load"),
                            ("chain_head_kernel", (128, 4), "buffer_store")):
        ins = kernels[name, par]
        found = 0
        for i, (a, s, t) in enumerate(ins):
            if s.startswith(pick) and not s.endswith(" lds"):
                try:
                    check(name, par, ins[:i] + [(a, "s_nop 0", t)] + ins[i + 1:])
                except AssertionError:
                    found += 1
        assert found, (name, par, pick)
