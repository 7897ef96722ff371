"""What bench.py makes of a counter summary."""
import sys
from pathlib import Path

ROOT = Path(__file__).resolve().parents[1]


def test_matrix_instructions_take_sixteen_cycles():
    sys.path.insert(0, str(ROOT))
    import bench
    assert bench.vector_pipe_cycles({"SQ_INSTS_VALU": 1000.0}) == 4000.0
    assert bench.vector_pipe_cycles({"SQ_INSTS_VALU": 1000.0, "SQ_INSTS_MFMA": 100.0}) == 900 * 4 + 100 * 16
