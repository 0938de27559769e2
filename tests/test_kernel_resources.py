"""Build-time check of the registers and the LDS the compiler gives the block and segment kernels (CPU only: hipcc
cross-compiles).

The headline kernel keeps 64 state registers per lane and runs four waves per SIMD, so it sits at the
128-register limit: a change that pushes more values into scratch memory inside the token loop would cost time on
every block without failing any numerical test.  (16 registers of a lane spill there now, 20 bytes, which caches
hold: traffic is 1.013 times the algorithmic one.)  The compiler's own resource remarks are parsed here."""
import os
import re
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_2605_11196_amd import build

CSRC = os.path.join(os.path.dirname(os.path.abspath(build.__file__)), "csrc")
LDS = 160 * 1024   # of a compute unit


def _value(x):
    x = x.strip()
    return {"true": True, "false": False, "float": "f32", "unsigned short": "bf16"}.get(x) if not x.isdigit() else int(x)


@pytest.fixture(scope="module")
def usage():
    """{kernel: {template arguments: resources}} of the sources with block and segment kernels"""
    sources = ["vla_chunk.hip", "vla_chunk_pipe.hip", "vla_chunk_d16.hip", "vla_chunk_general.hip", "vla_chunk_general_pipe.hip",
               "vla_two_phase.hip", "vla_a_map.hip", "vla_segments.hip"]
    with ThreadPoolExecutor(len(sources)) as pool:
        reports = list(pool.map(lambda f: build.resource_usage(os.path.join(CSRC, f)), sources))
    out = {}
    for report in reports:
        for name, r in report.items():
            m = re.search(r"(\w+)<([^>]*)>", name)
            if m:
                out.setdefault(m.group(1), {})[tuple(_value(x) for x in m.group(2).split(","))] = r
    return out


@pytest.fixture(scope="module")
def chunk_usage(usage):
    """the block kernel with one workgroup per head by (d_k, d_v, waves, io, feature map, split products)"""
    return {k[:6]: r for k, r in usage["chunk_kernel"].items() if not k[6]}


SQUARE_WAVES = [(16, 1), (32, 1), (64, 4), (96, 3), (128, 4)]   # d = 64, 128: three operand terms only


def test_every_block_kernel_instantiation_is_reported(chunk_usage):
    for d, nw in SQUARE_WAVES:
        for io in ("bf16", "f32"):
            for fmap in (False, True):
                one_term = io == "bf16" and not fmap
                if d not in (64, 128) or not one_term:
                    assert (d, d, nw, io, fmap, d > 16) in chunk_usage


@pytest.mark.parametrize("io", ["bf16", "f32"])
@pytest.mark.parametrize("d,nw", SQUARE_WAVES)
def test_block_kernels_use_no_scratch_and_keep_two_waves_per_simd(chunk_usage, d, nw, io):
    """Square heads, with waves of 32 and of 16 columns."""
    for fmap in (False, True):
        if (d, d, nw, io, fmap, d > 16) not in chunk_usage:
            continue
        r = chunk_usage[(d, d, nw, io, fmap, d > 16)]
        assert r["ScratchSize"] == 0 and r["VGPRSpill"] == 0, r
        assert r["VGPRs"] + r.get("AGPRs", 0) <= 256 and r["Occupancy"] >= 2, r


def test_headline_kernel_fits_two_workgroups_per_compute_unit(usage):
    r = usage["chunk_pipe_kernel"][(128, 128, 4, 4, "bf16", False, 4)]
    assert 2 * r["LDSSize"] <= LDS and r["Occupancy"] >= 4, r


def test_two_chain_kernels_hold_the_workgroups_they_are_chosen_for(usage):
    """(d_k, d_v, waves on A, waves on S): workgroups of a compute unit with one operand term and with three"""
    for (d, d_v, na, ns), held in {(64, 64, 2, 2): (4, None), (64, 64, 4, 4): (2, 2), (64, 16, 4, 1): (2, 1),
                                   (64, 128, 4, 8): (1, 1), (32, 32, 2, 2): (4, 4), (32, 96, 2, 6): (2, 2),
                                   (32, 128, 2, 8): (1, 1), (96, 96, 6, 6): (1, 1), (128, 128, 8, 8): (1, 1)}.items():
        for io, fmap, n in (("bf16", False, held[0]), ("bf16", True, held[1]), ("f32", False, held[1]), ("f32", True, held[1])):
            if n:
                r = next(r for k, r in usage["chunk_pipe_kernel"].items() if k[:6] == (d, d_v, na, ns, io, fmap))
                assert n * r["LDSSize"] <= LDS and n * (na + ns) <= 4 * r["Occupancy"], r


# Known scratch use, in bytes per lane and spilled registers; every other instantiation has none.
#   chunk_kernel: (d_k, d_v, waves, io, feature map, split products, heads in turn)
#   chunk_pipe_kernel: (d_k, d_v, waves on A, waves on S, io, feature map, waves per SIMD)
#   chunk_general_kernel: (d_k, d_v, columns of a wave, io, two sweeps, A chain alone, double buffers, split products)
#   chunk_general_pipe_kernel: (d_k, d_v, waves on A, waves on S, io, kind of u, waves per SIMD)
#   a_map_kernel: (d_k, waves on A, waves on the map, slots of a map wave, io, operand terms, waves per SIMD)
#   s_rows_lds_kernel: (d_k, tile slots, other value head size, io, maps, terms, split products, waves per SIMD)
KNOWN = {
    "chunk_kernel": {
        (96, 128, 3, "bf16", False, True, False): (20, 4),
    },
    "chunk_pipe_kernel": {
        (128, 128, 4, 4, "bf16", False, 4): (20, 16),
    },
    "chunk_general_kernel": {
        (32, 128, 16, "f32", True, False, False, True): (8, 1),
    },
    "chunk_general_pipe_kernel": {
        (128, 128, 4, 4, "bf16", 1, 4): (56, 51),
        (128, 16, 8, 1, "f32", 0, 3): (168, 65), (128, 16, 8, 1, "f32", 1, 3): (308, 205), (128, 16, 8, 1, "f32", 2, 3): (168, 65),
        (128, 16, 8, 1, "bf16", 0, 3): (44, 10), (128, 16, 8, 1, "bf16", 1, 3): (120, 41), (128, 16, 8, 1, "bf16", 2, 3): (28, 6),
    },
    "a_map_kernel": {
        (32, 2, 2, 5, "f32", 3, 4): (48, 40), (32, 2, 2, 5, "bf16", 1, 4): (36, 21), (32, 2, 2, 5, "bf16", 3, 4): (32, 20),
        (64, 4, 4, 3, "f32", 3, 4): (28, 28), (64, 4, 4, 3, "bf16", 1, 4): (16, 10), (64, 4, 4, 3, "bf16", 3, 4): (24, 18),
        (96, 6, 6, 3, "f32", 3, 3): (8, 1), (96, 6, 6, 3, "bf16", 1, 3): (20, 16),
    },
    "gram_fixed_kernel": {
        (64, "f32"): (104, 57), (64, "bf16"): (24, 5),
        (128, "f32"): (140, 124), (128, "bf16"): (16, 5), (96, "f32"): (24, 9),
    },
    "gram_kernel": {}, "gram_given_a0_kernel": {}, "boundary_kernel": {},
    "combine_kernel": {},
    "chunk_d16_kernel": {},
    "a_scan_kernel": {},
    "s_rows_lds_kernel": {
        (128, 1, False, "f32", False, 3, True, 4): (96, 35), (128, 1, False, "f32", True, 3, True, 4): (20, 8),
        (128, 1, False, "bf16", False, 1, True, 4): (36, 20), (128, 1, False, "bf16", False, 3, True, 4): (60, 26),
        (128, 1, False, "bf16", True, 3, True, 4): (20, 8),
        (128, 1, True, "f32", False, 3, True, 4): (104, 37), (128, 1, True, "f32", True, 3, True, 4): (20, 8),
        (128, 1, True, "bf16", False, 1, True, 4): (24, 9), (128, 1, True, "bf16", False, 3, True, 4): (56, 25),
        (128, 1, True, "bf16", True, 1, True, 4): (20, 8), (128, 1, True, "bf16", True, 3, True, 4): (20, 8),
        (32, 4, True, "f32", False, 3, True, 2): (64, 23), (32, 4, True, "bf16", False, 1, True, 2): (20, 8),
        (32, 4, True, "bf16", False, 3, True, 2): (20, 8),
        (96, 1, False, "bf16", False, 1, True, 4): (20, 8), (96, 1, True, "bf16", False, 1, True, 4): (20, 8),
        (96, 2, True, "f32", False, 3, True, 2): (20, 8), (96, 2, True, "f32", True, 3, True, 2): (20, 8),
        (96, 2, True, "bf16", True, 3, True, 2): (20, 8),
    },
}


@pytest.mark.parametrize("kernel", sorted(KNOWN))
def test_no_kernel_exceeds_its_known_scratch_use(usage, kernel):
    assert usage[kernel], kernel
    over = {args: (r["ScratchSize"], r["VGPRSpill"]) for args, r in usage[kernel].items()
            if (r["ScratchSize"], r["VGPRSpill"]) > KNOWN[kernel].get(args, (0, 0))}
    assert not over, over


def test_no_boundary_workgroup_has_an_odd_number_of_waves(usage):
    """They would put the two waves of the workgroups that follow, those of the option kernel's A chain of heads of 32, on
    other SIMDs than those they share two and two, which costs that kernel a fifth of its time."""
    for args, r in usage["boundary_kernel"].items():
        assert r["Threads"] % 128 == 0, (args, r)


@pytest.mark.parametrize("io", ["bf16", "f32"])
def test_option_a_chain_leaves_room_for_the_workgroups_of_a_segment_plan(usage, io):
    """With options, heads of 64 are planned as 768 (head, segment) pairs, one round of three workgroups per compute unit,
    and heads of 32 as 1024."""
    for d, workgroups in ((64, 3), (32, 4)):
        for full in (True, False):
            r = usage["chunk_general_kernel"][(d, d, 16, io, full, True, True, False)]
            assert workgroups * r["LDSSize"] <= LDS, r
            assert workgroups * d // 16 <= 4 * r["Occupancy"], r


@pytest.mark.parametrize("d,d_v,nw,workgroups", [(64, 16, 2, 4), (64, 32, 2, 4), (64, 96, 2, 4), (64, 128, 2, 4),
                                                 (32, 16, 1, 8), (32, 64, 1, 8)])
def test_unsplit_kernels_hold_the_workgroups_they_are_chosen_for(chunk_usage, d, d_v, nw, workgroups):
    for io, fmap in (("f32", False), ("f32", True), ("bf16", True)):
        r = chunk_usage[(d, d_v, nw, io, fmap, False)]
        assert workgroups * r["LDSSize"] <= LDS, r
        assert workgroups * nw <= 4 * r["Occupancy"], r
