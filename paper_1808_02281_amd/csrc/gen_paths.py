"""Generate ``path_table.hpp``: the 34 Symanzik loops and, per link direction, the 48
staples the force sums (arXiv:1808.02281, Sec. II, eq. 18_3_27_30 and the force
algorithm after eq. 18_6_6_13).

Run at build time. Every staple is emitted as the path from site k+rho back to site k
(signed directions, +-(axis+1)), so that U_{k,rho} times the staple is the loop
rotated to start on link (k,rho):

* a loop position l with d_l = +rho gives the path d_{l+1} .. d_L, d_1 .. d_{l-1};
* a loop position l with d_l = -rho gives the reversed loop's path
  -d_{l-1} .. -d_1, -d_L .. -d_{l+1}.

Staples are grouped by class (plaquette, rectangle, cube) so that kernels can sum
each class separately.
"""
import itertools
import os
import sys

CLASS_NAMES = ("plaquette", "rectangle", "cube")


def loops():
    """The 34 direction sequences per site: (class, dirs)."""
    out = []
    for m, n in itertools.combinations(range(1, 5), 2):
        out.append((0, (m, n, -m, -n)))
    for m, n in itertools.permutations(range(1, 5), 2):
        out.append((1, (m, m, n, -m, -m, -n)))
    for m, n, r in itertools.combinations(range(1, 5), 3):
        for sn, sr in itertools.product((1, -1), repeat=2):
            out.append((2, (m, sn * n, sr * r, -m, -sn * n, -sr * r)))
    return out


def staples(rho):
    """The 48 staples of link direction rho (1-based axis), as (class, path) sorted by class."""
    res = []
    for cls, d in loops():
        L = len(d)
        for l in range(L):
            if d[l] == rho:
                path = d[l + 1:] + d[:l]
            elif d[l] == -rho:
                path = tuple(-x for x in reversed(d[:l])) + tuple(-x for x in reversed(d[l + 1:]))
            else:
                continue
            res.append((cls, path))
    res.sort(key=lambda s: s[0])
    return res


def check(rho, st):
    counts = [sum(1 for c, _ in st if c == k) for k in range(3)]
    assert counts == [6, 18, 24], counts
    for _, path in st:
        disp = [0, 0, 0, 0]
        disp[rho - 1] = 1  # start at k + rho
        for s in path:
            disp[abs(s) - 1] += 1 if s > 0 else -1
        assert disp == [0, 0, 0, 0], "staple must end at k"


def render():
    lines = [
        "// Generated by gen_paths.py; do not edit.",
        "// Staples of the one-loop Symanzik gauge force, arXiv:1808.02281 Sec. II:",
        "// for link direction rho (0..3), 48 paths from site k+rho back to site k, as signed",
        "// directions +-(axis+1); 6 plaquette, then 18 rectangle, then 24 cube staples.",
        "#pragma once",
        "",
        "namespace sym {",
        "namespace table {",
        "",
        "constexpr int kStaples = 48;",
        "constexpr int kClassBegin[4] = {0, 6, 24, 48};",
        "",
        "struct StapleDef {",
        "  int cls;",
        "  int len;",
        "  int dir[5];",
        "};",
        "",
        "constexpr StapleDef kStaple[4][48] = {",
    ]
    for rho in range(1, 5):
        st = staples(rho)
        check(rho, st)
        lines.append("  {")
        for cls, path in st:
            dirs = list(path) + [0] * (5 - len(path))
            lines.append("    {%d, %d, {%s}},  // %s" % (cls, len(path), ", ".join("%2d" % v for v in dirs),
                                                         CLASS_NAMES[cls]))
        lines.append("  },")
    lines += ["};", "", "}  // namespace table", "}  // namespace sym", ""]
    return "\n".join(lines)


def main(out_path=None):
    here = os.path.dirname(os.path.abspath(__file__))
    out_path = out_path or os.path.join(here, "path_table.hpp")
    text = render()
    old = open(out_path).read() if os.path.exists(out_path) else None
    if old != text:
        with open(out_path, "w") as f:
            f.write(text)
    return out_path


if __name__ == "__main__":
    print(main(sys.argv[1] if len(sys.argv) > 1 else None))
