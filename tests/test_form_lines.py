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


def test_fp32_scores_of_a_batch(tmp_path):
    # (entries, units) over all models: us of a call with waves of two row pairs, us with bands
    measured = {(96, 656): (70, 109), (192, 1312): (110, 123), (384, 2624): (192, 165), (660, 4510): (323, 255),
                (500, 1500): (170, 150), (750, 2250): (274, 216), (140, 1540): (123, 149), (420, 4620): (253, 233),
                (560, 6160): (322, 275), (192, 4480): (208, 383), (384, 8960): (361, 446), (576, 13440): (511, 527),
                (960, 22400): (803, 676), (336, 10640): (370, 476), (672, 21280): (662, 711), (672, 29274): (930, 1012),
                # 8 models
                (768, 5248): (244, 198), (1536, 10496): (423, 288), (1536, 35840): (958, 807)}
    holds(tmp_path, *(f"score32_wave_pairs({n}, {u}, 0) == {2 if waves < bands else 0}"
                      for (n, u), (waves, bands) in measured.items()),
          # one row pair: 21 entries 30 us, 44 with two; 32 entries 72 and 85
          "score32_wave_pairs(21, 665, 0) == 1", "score32_wave_pairs(32, 1280, 0) == 1",
          # the cap: 168 entries of 4 workgroups
          "score32_wave_pairs(168, 5320, 672) == 2", "score32_wave_pairs(168, 5320, 671) == 0",
          "score32_wave_pairs(10, 300, 80) == 1", "score32_wave_pairs(10, 300, 79) == 0")


def test_features_of_one_image(tmp_path):
    # strip rows: us by a wave per cell row, us in strips
    cell_map = {2160: (84, 185), 3456: (120, 184), 3960: (136, 184), 4400: (151, 184), 4950: (168, 184), 5850: (200, 184),
                6144: (199, 184), 6656: (218, 185), 8640: (288, 235), 9775: (329, 247), 10240: (333, 237)}
    plain = {3960: (56, 141), 6656: (88, 141), 8640: (114, 183), 10240: (109, 185)}
    holds(tmp_path, *(f"{n} {'<=' if rows < strips else '>'} FR_MAX_ROWS_CM_ONE" for n, (rows, strips) in cell_map.items()),
          *(f"{n} {'<=' if rows < strips else '>'} FR_MAX_ROWS" for n, (rows, strips) in plain.items()))
