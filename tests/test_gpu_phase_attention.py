"""The per-phase attention over query tiles that share rows, at the sizes where its plan can go wrong, against the fp64
oracle: two to seven query tiles (one group and two), cached rows at and past the 32 of a tile and the two tiles of a
step, empty agents, one chunk and several, rings that wrap, both layouts, bf16 and fp8; a shared cache whose agents start
at one slot (their query tiles share workgroups) and at different ones (they do not).  Keys are of the kind that moves a
query's running maximum (outlier channels, a growing scale, a sink row), so that a wrong row shows.  Tolerances as in the
parity tests: 2e-2 of the largest value, the bf16 rounding of 2 layers' operands."""

from __future__ import annotations

import numpy as np
import pytest
import torch

import synth
from harness import Cache, Model, record, rel_err, run_forward, tokens_for
from paper_2607_15621_amd import fsx

pytestmark = pytest.mark.gpu

TOL = 2e-2


def workload(name, wid, lengths, frame, cache="bf16", heads=8, capacity=None, stress=True):
    return synth.Workload(name=name, wid=wid, n_layers=2, d_model=256, n_heads=heads, head_dim=128, d_ffn=512,
                          n_expert_tokens=10, n_frame_tokens=frame, batch=len(lengths), lengths=tuple(lengths),
                          dtype="bf16", cache_dtype=cache, capacity=capacity or max(max(lengths), 1) + 3,
                          stress_keys=stress)


# frame tokens, lengths, cache dtype, token-major
CASES = [(7, (0, 1, 33), "bf16", False), (23, (31, 32, 64, 65), "fp8", True), (87, (700, 0, 95), "bf16", True),
         (95, (2100,), "bf16", False), (64, (1500, 40), "fp8", False), (6, (5000,), "fp8", True)]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_query_tiles_sharing_rows_match_oracle(case):
    frame, lengths, cache_dtype, token_major = CASES[case]
    print(f"case phase attention {CASES[case]}", flush=True)
    wl = workload(f"phatt{case}", 760 + case, lengths, frame, cache_dtype, heads=2 if max(lengths) > 1000 else 8)
    model = Model(wl)
    ex = model.create(flags=fsx.FLAG_MULTI_LAUNCH)
    cache = Cache(wl, starts=[(wl.capacity - 5 + 3 * b) % wl.capacity for b in range(wl.batch)],
                  layout=fsx.CACHE_TOKEN_MAJOR if token_major else fsx.CACHE_HEAD_MAJOR)
    host_tok, tok = tokens_for(wl)
    wp, hid = run_forward(ex, cache, tok, wl.batch, frame, with_hidden=True)
    for b in range(wl.batch):
        ref_wp, ref_hid = model.oracle_agent(host_tok[b], cache.oracle_rows(b, decoded=True), cache.desc.pos[b])
        record(b, rel_err(wp[b], ref_wp), TOL)
        record(b, max(rel_err(hid[l, b], ref_hid[l]) for l in range(wl.n_layers)), TOL, what="worst layer hidden")
    wp2, hid2 = run_forward(ex, cache, tok, wl.batch, frame, with_hidden=True)
    assert np.array_equal(wp, wp2) and np.array_equal(hid, hid2), "two forwards differ bitwise"
    ex.close()


@pytest.mark.parametrize("flags", [0, fsx.FLAG_MULTI_LAUNCH])
@pytest.mark.parametrize("starts_differ,frame,rows", [(False, 0, 170), (False, 20, 64), (True, 0, 170), (False, 0, 3000)])
def test_agents_of_a_shared_cache_match_oracle(flags, starts_differ, frame, rows):
    """Agent j sees the first lens[j] rows from its start: some none, some a part of the longest agent's last tile."""
    print(f"case shared attention {flags} {starts_differ} {frame} {rows}", flush=True)
    lens = [rows, 0, rows // 2 + 1, 32, rows - 1, 33, 1]
    starts = [5 * j if starts_differ else 9 for j in range(len(lens))]
    wl = workload("phshared", 780, lens, frame, capacity=rows + 40, heads=8)
    model = Model(wl)
    ex = model.create(flags=flags)
    full = Cache(wl.replace(batch=1, lengths=(rows + 40,)))  # every slot of the ring holds a row
    desc = fsx.CacheDesc(full.k, full.v, fsx.BF16, wl.n_layers, wl.n_heads, wl.head_dim, wl.capacity, lens, positions=lens,
                         starts=starts, layout=fsx.CACHE_SHARED)
    host_tok, tok = tokens_for(wl)
    n = len(lens)
    wp = torch.full((n, wl.n_out), float("nan"), device="cuda")
    fsx.expert_forward(ex, desc, tok, n, frame, wp, None)
    torch.cuda.synchronize()
    slab = full.oracle_rows(0)
    for j in range(n):
        slots = (starts[j] + np.arange(lens[j])) % wl.capacity
        ref, _ = model.oracle_agent(host_tok[j], lambda l: tuple(x[slots] for x in slab(l)), lens[j])
        record(j, rel_err(wp[j].cpu().numpy(), ref), TOL)
    if rows == 170 and not starts_differ:  # what only the longest agent sees does not reach the others
        full.k[:, :, :, (9 + rows - 1) % wl.capacity] = float("nan")
        full.v[:, :, :, (9 + rows - 1) % wl.capacity] = float("nan")
        wp2 = torch.zeros_like(wp)
        fsx.expert_forward(ex, desc, tok, n, frame, wp2, None)
        torch.cuda.synchronize()
        assert torch.isnan(wp2[0]).all() and torch.equal(wp2[1:], wp[1:])
    ex.close()


def check_route(wl, make_desc, phases, what):
    """The default handle takes the faster form, bit for bit, and so does the allocation-free entry point."""
    model = Model(wl)
    desc = make_desc()
    host_tok, tok = tokens_for(wl)
    shapes = (wl.batch, wl.n_out), (wl.n_layers, wl.batch, wl.seq, wl.d_model)
    got = {}
    for name, flags in (("default", 0), ("phases", fsx.FLAG_MULTI_LAUNCH), ("kernel", fsx.FLAG_TRACE)):
        ex = model.create(flags=flags)
        calls = [(name, fsx.expert_forward)] + ([("noalloc", fsx.expert_forward_noalloc)] if name == "default" else [])
        for key, call in calls:
            wp, hid = (torch.full(s, float("nan"), device="cuda") for s in shapes)
            call(ex, desc, tok, wl.batch, wl.n_frame_tokens, wp, hid)
            torch.cuda.synchronize()
            got[key] = wp.cpu().numpy(), hid.cpu().numpy()
        ex.close()
    same = lambda a, b: all(np.array_equal(x, y) for x, y in zip(got[a], got[b]))  # noqa: E731
    assert not same("phases", "kernel"), "the two forms agree bitwise: the test could not tell them apart"
    assert same("default", "phases" if phases else "kernel"), what
    assert same("noalloc", "default")
    for x, y in zip(got["phases"], got["kernel"]):
        assert rel_err(x, y) <= TOL


# agents, frame tokens, cached rows of each, shared cache, whether a launch per phase is the faster form
ROUTES = [(1, 22, 1023, False, False), (1, 22, 1024, False, True), (1, 23, 40, False, True), (2, 7, 40, False, True),
          (9, 0, 40, False, False), (10, 0, 40, False, True), (10, 0, 820, False, False), (15, 0, 820, False, True),
          (9, 0, 40, True, False), (10, 0, 40, True, True)]


@pytest.mark.parametrize("batch,frame,rows,shared,phases", ROUTES)
def test_route_of_a_tick_by_its_rows(batch, frame, rows, shared, phases):
    """Both sides of every line over the rows of tokens."""
    print(f"case route {batch} {frame} {rows} {shared}", flush=True)
    wl = workload("phroute", 790, (rows,) * batch, frame, heads=2)
    cache = Cache(wl.replace(batch=1, lengths=(rows,)) if shared else wl)
    if shared:
        cache.desc = fsx.CacheDesc(cache.k, cache.v, fsx.BF16, wl.n_layers, wl.n_heads, wl.head_dim, wl.capacity,
                                   [rows] * batch, positions=[rows] * batch, layout=fsx.CACHE_SHARED)
    check_route(wl, lambda: cache.desc, phases, "the other form was taken")


# agents, frame tokens, cached rows of each, fp8 cache, whether a launch per phase is the faster form: 32 heads, histories on
# both sides of where the kernel's streaming makes up for its rounds
LONG_ROUTES = [(15, 0, 1066, False, True), (15, 0, 1067, False, False), (15, 0, 1866, True, True), (15, 0, 1867, True, False),
               (16, 0, 3751, False, True), (16, 0, 3750, True, True), (16, 0, 3751, True, False),
               (1, 22, 12000, True, True), (1, 22, 12001, True, False), (1, 22, 12001, False, True),
               (1, 30, 223, False, False), (1, 30, 224, False, True)]


@pytest.mark.parametrize("batch,frame,rows,fp8,phases", LONG_ROUTES)
def test_route_of_a_tick_by_its_history(batch, frame, rows, fp8, phases):
    print(f"case route of 32 heads {batch} {frame} {rows} {fp8}", flush=True)
    wl = workload("phlong", 791, (rows,) * batch, frame, "fp8" if fp8 else "bf16", heads=32)
    shape = (batch, wl.n_layers, wl.n_heads, wl.capacity, wl.head_dim)
    g = torch.Generator(device="cuda").manual_seed(791)

    def desc():
        k, v = (torch.randn(shape, generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(2))
        if not fp8:
            return fsx.CacheDesc(k, v, fsx.BF16, wl.n_layers, wl.n_heads, wl.head_dim, wl.capacity, wl.lengths)
        k, v = (x.to(torch.float8_e4m3fn).view(torch.uint8) for x in (k, v))
        ones = torch.ones(shape[:3], device="cuda")
        return fsx.CacheDesc(k, v, fsx.FP8_E4M3, wl.n_layers, wl.n_heads, wl.head_dim, wl.capacity, wl.lengths, k_scale=ones,
                             v_scale=ones)

    check_route(wl, desc, phases, "the other form was taken")
