"""Layout of Stage 3's workspaces: buffers disjoint, inside the size that the
library asks for, and the rotation log (stored and loaded 16 bytes at a time) on
a 16-byte boundary."""
import random

from host_rules import run_program
from paper_2608_07814_amd import lorex as lx

BODY = """
    long rows, cols, np, l;
    std::cin >> rows >> cols >> np >> l;
    const lx::Stage3Ws w = lx::stage3_ws(rows, cols, np, l);
    std::printf("%ld %ld %ld %ld %ld %ld %ld %ld %ld %ld %ld %ld %ld %ld %ld %ld\\n", (long)w.R, (long)w.Xp, (long)w.P,
                (long)w.Y, (long)w.Z, (long)w.T, (long)w.Wt, (long)w.G, (long)w.U, (long)w.Ve, (long)w.lam,
                (long)w.sig, (long)w.Ad, (long)w.part, (long)w.total, (long)lx::kDgParts);
"""


def test_layout(tmp_path):
    rng = random.Random(3)
    cases = [(17, 33, -1, 1), (17, 33, 4, 1), (3, 3, -1, 3), (2048, 768, -1, 74), (2048, 768, 3000, 74),
             (129, 1001, 177, 128)]
    while len(cases) < 60:
        rows, cols = rng.randint(1, 300), rng.randint(1, 300)
        l = rng.randint(1, min(rows, cols, 128))
        cases.append((rows, cols, rng.choice((-1, l, l + rng.randint(0, 400))), l))
    L = lx.lib()
    odd = 0
    for (rows, cols, np_, l), row in zip(cases, run_program(tmp_path, "lx_stage3_ws.h", BODY, cases)):
        *at, part, total, parts = map(int, row)
        lp, w = l + (l & 1), np_ >= 0
        n = max(np_, 0)
        sizes = [rows * cols, n * cols, cols * l if w else 0, rows * l, (n if w else cols) * l, l * cols, l * n,
                 lp * lp, lp * lp, lp * lp, lp, lp, rows * l]
        end = 0
        for a, size in zip(at, sizes):
            assert a >= end
            end = a + size
        assert part >= end and part % 2 == 0 and part + parts <= total
        odd += end % 2
        want = (L.lx_weighted_workspace_bytes(rows, cols, np_, 0, l, 0) if w
                else L.lx_lowrank_workspace_bytes(rows, cols, l, 0))
        assert want == 8 * total
        assert total == sum(sizes) + lp * lp + parts
    assert odd > 5
