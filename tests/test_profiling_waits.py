"""The table of what each kernel's waves do with their time, on a hand-made counter run."""

import csv

from paper_2208_12569_amd import profiling


def test_shares_of_a_wave_s_time(tmp_path):
    path = tmp_path / "w.csv"
    runs = {"void fq::(anonymous namespace)::a<float>(int)": [(1, 2.0), (2, 6.0)], "void fq::b": [(3, 1.0)], "other": [(4, 9.0)]}
    per_wave = {"SQ_WAVES": 1.0, "SQ_WAVE_CYCLES": 100.0, "SQ_WAIT_ANY": 50.0, "SQ_WAIT_INST_ANY": 20.0,
                "SQ_ACTIVE_INST_ANY": 30.0, "SQ_INSTS_VALU": 400.0, "SQ_ACTIVE_INST_VALU": 10.0,
                "SQ_THREAD_CYCLES_VALU": 480.0}
    with open(path, "w", newline="") as fh:
        w = csv.writer(fh)
        w.writerow(["Dispatch_Id", "Kernel_Name", "Counter_Name", "Counter_Value"])
        for name, launches in runs.items():
            for d, waves in launches:
                for c, v in per_wave.items():
                    w.writerow([d, name, c, v * waves / 2])  # two rows of a dispatch add up
                    w.writerow([d, name, c, v * waves / 2])
    rows = [r for r in profiling.waits_md(str(path), "cmd").splitlines() if r.startswith("| ")][1:]
    assert rows[0].startswith("| a<float>") and rows[0].endswith("| 2 | 4 | 400 | 48.0 | 0.30 | 0.20 | 0.50 |")
    assert len(rows) == 2 and rows[1] == "| fq::b | 1 | 1 | 400 | 48.0 | 0.30 | 0.20 | 0.50 |"
