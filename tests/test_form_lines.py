"""The lines between two forms of a stage, held against measurements on both
sides: the rules of the sources, compiled here, must pick the form that was
faster (no GPU)."""
import subprocess

from paper_1611_01642_amd import build


def holds(tmp_path, *claims):
    """Each claim, a constant expression over the sources' rules, is true."""
    src = tmp_path / "lines.hip"
    src.write_text('#include "pd_internal.h"\nusing namespace pd;\n' +
                   "".join(f'static_assert({c}, "{c}");\n' for c in claims))
    res = subprocess.run([build.hipcc(), "--offload-host-only", "-fsyntax-only", "-std=c++17", "-I", build.CSRC, str(src)],
                         capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr


def test_scores_of_one_image(tmp_path):
    # table entries over all models: us by waves, us on the vector ALUs
    measured = {64: (43, 376), 128: (83, 388), 256: (216, 379), 264: (269, 347), 288: (146, 375), 384: (322, 493),
                473: (430, 456), 512: (427, 495), 792: (695, 622), 992: (888, 779), 1056: (909, 787),
                2048: (2017, 1503), 2112: (1763, 1506)}
    holds(tmp_path, *(f"{'' if waves < valu else '!'}score_single_by_waves({n})" for n, (waves, valu) in measured.items()))
