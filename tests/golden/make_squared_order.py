"""Write squared_order.json: the checksums of tests/test_gpu_sq_bits.py, from the
library that PYTHONPATH puts first.  The file in the repository is from the library of
commit 095df9d (git worktree, build, run this with that tree first in PYTHONPATH)."""
import json
import sys
from pathlib import Path

HERE = Path(__file__).resolve().parent
sys.path.append(str(HERE.parents[1]))
sys.path.append(str(HERE.parent))

import paper_1205_2933_amd as mg  # noqa: E402
from test_gpu_sq_bits import CASES, results  # noqa: E402

if __name__ == "__main__":
    out = {}
    for name, case in CASES.items():
        out[name] = results(mg, case)
        print(name, out[name], flush=True)
    target = Path(sys.argv[1]) if len(sys.argv) > 1 else HERE / "squared_order.json"
    target.write_text(json.dumps(out, indent=1) + "\n")
