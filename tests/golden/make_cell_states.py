"""Writes ``cell_states.npz``: elements of the states that test_gpu_cell_states.py
compares, as the built library gives them on the GPU.  They were recorded with the
library whose cells ran every product, QR and rotation in the order that cells
with wide cuts keep.

Run: ``python tests/golden/make_cell_states.py [OUTPUT]``.
"""
import os
import sys

import numpy as np

HERE = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, os.path.dirname(HERE))
sys.path.insert(0, os.environ.get("SICTM_TREE", os.path.dirname(os.path.dirname(HERE))))

import test_gpu_cell_states as T  # noqa: E402

out = {}
for case in T.CASES:
    x = T.iterate(*case)
    out["_".join(map(str, case))] = x[T.places(x.size, case[5])]
    print(case, x.size, flush=True)
np.savez(sys.argv[1] if len(sys.argv) > 1 else os.path.join(HERE, "cell_states.npz"), **out)
