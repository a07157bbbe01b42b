"""The fp32 per-op kernels at the sizes where they can go wrong, every agent and layer against the fp64 oracle.

Widths that are no multiple of four (one element per load instead of four), widths past one staged chunk of 512
columns, heads past one block of output channels (64 or 256), rows past the eight of a workgroup, cached and own rows at
and past the 64 of an attention tile, empty and wrapping rings, every cache dtype, more pooled tokens than the head takes
at a time.  Tolerance: sums of up to 1,100 fp32 products over three layers, n eps / 2 in the worst case and about
sqrt(n) eps = 2e-6 relative for random signs; 1e-5 of the largest value is five times that.
"""

from __future__ import annotations

import numpy as np
import pytest

import synth
from harness import Cache, Model, record, rel_err, run_forward, tokens_for
from paper_2607_15621_amd import fsx

pytestmark = pytest.mark.gpu

TOL = 1e-5

# d, heads, head_dim, ffn, expert tokens, frame tokens, lengths, cache dtype, token-major
CASES = [
    (33, 3, 6, 50, 3, 2, (0, 5, 70), "f32", False),
    (520, 2, 130, 36, 9, 0, (64, 65), "bf16", True),
    (48, 2, 260, 1030, 17, 50, (63, 129, 300), "fp8", False),
    (34, 5, 2, 7, 1, 0, (257,), "fp8", True),
    (516, 4, 64, 132, 8, 0, (1, 1000), "f32", True),
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_fp32_expert_of_odd_sizes_matches_oracle(case):
    d, H, Dh, F, T, frame, lengths, cache_dtype, token_major = CASES[case]
    print(f"case per-op {CASES[case]}", flush=True)
    cap = max(lengths) + 3
    wl = synth.Workload(name=f"per_op{case}", wid=700 + case, n_layers=3, d_model=d, n_heads=H, head_dim=Dh, d_ffn=F,
                        n_expert_tokens=T, n_frame_tokens=frame, batch=len(lengths), lengths=lengths, dtype="f32",
                        cache_dtype=cache_dtype, capacity=cap)
    model = Model(wl)
    ex = model.create()
    assert fsx.expert_info(ex)["path"] == 1
    cache = Cache(wl, starts=[(cap - 2 + 7 * b) % cap for b in range(wl.batch)],
                  layout=fsx.CACHE_TOKEN_MAJOR if token_major else fsx.CACHE_HEAD_MAJOR)
    host_tok, tok = tokens_for(wl)
    wp, hid = run_forward(ex, cache, tok, wl.batch, frame, with_hidden=True)
    for b in range(wl.batch):
        ref_wp, ref_hid = model.oracle_agent(host_tok[b], cache.oracle_rows(b, decoded=True), cache.desc.pos[b])
        record(b, rel_err(wp[b], ref_wp), TOL)
        record(b, max(rel_err(hid[l, b], ref_hid[l]) for l in range(wl.n_layers)), TOL, what="worst layer hidden")
    assert np.array_equal(wp, run_forward(ex, cache, tok, wl.batch, frame)[0]), "two forwards differ bitwise"
    ex.close()
