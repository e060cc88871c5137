"""What the benchmark's line says of its sample counts: the timed renders step
over samples that the counts and the ALU roofline made of them include, so
every such roofline carries the statement."""
import re

import bench


def test_rooflines_say_what_they_count():
    lines = bench.rooflines(1e9, 31, 1e8, 1e-3)
    alu = [r for r in lines if r["bound"] == "alu"]
    assert len(alu) == 1 and "step" in alu[0]["samples_counted"]
    src = open(bench.__file__).read()
    made = re.findall(r'\{"bound": "alu".*?\}', src, flags=re.S)
    assert len(made) >= 5 and all("samples_counted" in m for m in made)
