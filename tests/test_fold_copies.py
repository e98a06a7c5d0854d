"""The folded iteration's scalars (csrc/recurrence.h): a launch whose blocks copy a
right-hand side's scalars never writes that copy, so no block reads what another
writes.  Checked on the source: every fold reads through a pointer to const and
stores only to its second pointer, and the launches pass different copies."""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2602_14450_amd", "csrc")


def source(name):
    text = open(os.path.join(CSRC, name)).read()
    return re.sub(r"//[^\n]*", "", text)


def test_folds_write_another_copy_than_they_read():
    text = source("recurrence.h")
    assert "const_cast" not in text
    folds = re.findall(r"void (fold_\w+)\(Scalars& sh, ((?:const )?Scalars\*) (\w+), (\w+[^)]*)\) \{(.*?)\n\}", text, re.S)
    assert {f[0] for f in folds} == {"fold_iter_end", "fold_alpha", "fold_omega"}
    for name, kind, src, rest, body in folds:
        assert kind == "const Scalars*", name
        dst = re.match(r"Scalars\* (\w+)", rest).group(1)
        assert dst != src and f"copy_scalars({dst} + rhs, &sh)" in body, name
        assert not re.search(rf"=\s*{src}\s*\+|{src}(\[\w+\]|->)", body), name


def test_launches_pass_two_copies():
    blas, op = source("blas.hip"), source("dslash.hip")
    flat = lambda s: re.sub(r"\s+", " ", s)  # noqa: E731
    read_write = {"p": r"k_p_update<S, true>\).*?, g, (f\.\w+), (f\.\w+),",
                  "s": r"k_s_update<S, true>\).*?, g, (f\.\w+), (f\.\w+),",
                  "xr": r"k_xr_update<S, true>\).*?, g, (f\.\w+), (f\.\w+),"}
    want = {"p": ("f.sc", "f.next"), "s": ("f.next", "f.mid"), "xr": ("f.mid", "f.sc")}
    for k, pattern in read_write.items():
        assert re.search(pattern, flat(blas)).groups() == want[k], k
    for name, pair in (("hp", want["p"]), ("hs", want["s"])):
        got = re.search(rf"SplitSrc<S> {name}\{{\w+, v, nullptr, (f\.\w+), (f\.\w+),", flat(op))
        assert got.groups() == pair, name
