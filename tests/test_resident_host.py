"""resident_steps reads its instance from and writes it to the same memory in runs of an even number of steps; a restrict
qualifier on either pointer would promise the compiler that it does not, whatever it makes of that today."""
import pathlib
import re

SOURCE = pathlib.Path(__file__).resolve().parent.parent / "paper_2002_05265_amd" / "csrc" / "lbm_batch_resident.hpp"


def test_in_place_runs_make_no_aliasing_promise():
    text = SOURCE.read_text()
    assert "(n + nsteps) & 1" in text  # the copy it ends in: the one it starts from for an even number
    params = re.search(r"void resident_steps\((.*?)\)\s*\{", text, re.S).group(1)
    for name in ("src", "dst"):
        (decl,) = [p for p in params.split(",") if re.search(rf"\b{name}$", p.strip())]
        assert "restrict" not in decl, decl
