"""GPU parity of the time-parallel mode: segments of the sequence run concurrently from boundary states
(A from the explicit inverse of Section 3.2 in float64, S from composed per-segment affine maps of
eq. (s-update)); the result must match the sequential fp64 oracle to the same tolerance as every other mode.
"""
import numpy as np
import pytest

import oracle
import vla_inputs
from parity_utils import TOL, check_parity, gpu_forward, slab_rel_err

pytestmark = pytest.mark.gpu

TP = 4  # VLA_MODE_TIME_PARALLEL


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d,T,segments", [
    (64, 1000, 5),      # ragged: 63 blocks in segments of 13, the last one short, last block 8 tokens
    (32, 200, 256),     # more segments asked for than blocks: one block per segment
    (128, 513, 2),      # second segment ends in a one-token block
    (128, 300, 7),
    (96, 700, 6),       # three waves per head, keys staged by 6 threads of 16 elements; Gram sums and the
    (96, 47, 3),        # boundary inverse run in the d = 128 layout with the extra columns held at zero
    (64, 4096, 0),      # the library's own choice (16 segments for 6 heads)
    (32, 2048, 0),
    (64, 16, 4),        # a single block: degenerates to one segment
])
def test_segments_match_the_sequential_oracle(d, T, segments, dtype):
    q, k, v = vla_inputs.gaussian_qkv(2, 3, T, d, seed=900 + d + T)
    errs, _, _ = check_parity(q, k, v, dtype=dtype, lambda0=0.1, mode=TP, segments=segments)
    print(d, T, segments, dtype, errs)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d,T,segments", [(64, 250, 8), (32, 300, 8), (128, 150, 8), (64, 16 * 9, 9), (96, 200, 8)])
def test_many_head_segment_pairs_take_the_shared_operand_kernels(d, T, segments, dtype):
    """32 heads x 8 segments = 256 (head, segment) pairs: from there on the S recurrence runs with one
    workgroup per pair and the block operands staged once through LDS (ragged last block, one- and
    two-block segments, the three-stage ring wrapping round)."""
    q, k, v = vla_inputs.gaussian_qkv(4, 8, T, d, seed=1200 + d + T)
    S0 = np.random.default_rng(d).standard_normal((4, 8, d, d)).astype(np.float32)
    errs, _, _ = check_parity(q, k, v, S0, None, dtype=dtype, lambda0=0.1, mode=TP, segments=segments)
    print(d, T, segments, dtype, errs)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d,T,segments", [(64, 300, 8), (32, 277, 8), (64, 16 * 8 + 1, 8), (32, 16 * 16, 8)])
def test_chip_filling_pair_counts_form_the_maps_inside_the_a_scan(d, T, segments, dtype):
    """96 heads x 8 segments = 768 (head, segment) pairs: from there on (d <= 64, no options) the A scan forms the
    per-segment affine maps of S itself, one block behind (two- and three-block segments, a ragged last block, a
    one-token last segment, a given S0 and A0)."""
    q, k, v = vla_inputs.gaussian_qkv(6, 16, T, d, seed=1250 + d + T)
    rng = np.random.default_rng(d + T)
    S0 = rng.standard_normal((6, 16, d, d)).astype(np.float32)
    R = rng.standard_normal((6, 16, d, d)) / np.sqrt(d)
    A0 = (np.eye(d) * 2.0 + R @ np.swapaxes(R, -1, -2)).astype(np.float32)   # symmetric positive definite
    A0 = (A0 + np.swapaxes(A0, -1, -2)) / 2
    errs, _, _ = check_parity(q, k, v, S0, A0, dtype=dtype, lambda0=0.1, mode=TP, segments=segments)
    print(d, T, segments, dtype, errs)


@pytest.mark.parametrize("d,T", [(64, 100), (128, 33), (32, 200), (96, 70)])
def test_two_phase_with_many_heads_takes_the_shared_operand_kernel(d, T):
    q, k, v = vla_inputs.gaussian_qkv(16, 16, T, d, seed=1300 + d)
    check_parity(q, k, v, lambda0=0.1, mode=3)


@pytest.mark.parametrize("d", [32, 64, 96, 128])
def test_given_initial_state_enters_the_boundary_inverse(d):
    """A non-trivial symmetric positive definite A0 and a non-zero S0 (the state after T1 tokens, from
    the oracle) must be carried through the boundary computation: A0 is inverted in float64 there."""
    T, T1 = 700, 123
    q, k, v = vla_inputs.gaussian_qkv(1, 4, T, d, seed=77 + d)
    full = oracle.forward(q, k, v, lambda0=0.1)
    head = oracle.forward(q[:, :, :T1], k[:, :, :T1], v[:, :, :T1], lambda0=0.1)
    o, S_T, A_T = gpu_forward(q[:, :, T1:], k[:, :, T1:], v[:, :, T1:], head["S_T"], head["A_T"],
                              mode=TP, segments=6)
    errs = dict(o=slab_rel_err(o, full["o"][:, :, T1:], 2), S=slab_rel_err(S_T, full["S_T"], 2),
                A=slab_rel_err(A_T, full["A_T"], 2))
    assert max(errs.values()) <= TOL["f32"], errs


@pytest.mark.parametrize("d", [32, 64, 96, 128])
@pytest.mark.parametrize("lambda0", [1e3, 1e6, 1e9, 1e30, float("inf")])
def test_boundary_inverse_of_large_elements(lambda0, d):
    """The block kernel is at 4e-7 and below over this range."""
    q, k, v = vla_inputs.gaussian_qkv(1, 3, 200, d, seed=80 + d)
    errs, _, _ = check_parity(q, k, v, lambda0=lambda0, mode=TP, segments=4, tol=1e-5)
    print(lambda0, d, errs)


@pytest.mark.parametrize("d", [32, 64, 96, 128])
@pytest.mark.parametrize("grades", [(-9, -9), (-8, 0)])
def test_given_initial_state_of_small_or_graded_elements(grades, d):
    """A0 with diagonal elements from 10^grades[0] to 10^grades[1], whose inverse has their reciprocals.  It is inverted twice,
    and A0 as small as 1e-9 passes both inverses all but unchanged."""
    q, k, v = vla_inputs.gaussian_qkv(1, 3, 200, d, seed=90 + d)
    R = np.random.default_rng(d).standard_normal((1, 3, d, d)) / np.sqrt(d)
    scale = 10.0 ** (0.5 * np.linspace(*grades, d))
    A0 = (scale[:, None] * (np.eye(d) + R @ np.swapaxes(R, -1, -2)) * scale).astype(np.float32)
    A0 = 0.5 * (A0 + np.swapaxes(A0, -1, -2))
    errs, _, _ = check_parity(q, k, v, None, A0, mode=TP, segments=4, tol=1e-5)
    print(grades, d, errs)


def test_recall_workload_with_zero_and_repeated_directions():
    """Mostly all-zero tokens and few distinct keys: the Gram sums are low-rank, so the boundary matrix
    lambda0 I + G has many eigenvalues equal to lambda0."""
    c = vla_inputs.CONFIGS["recall"]
    q, k, v, _ = vla_inputs.recall_task(4, c["H"], c["T"], c["d"], c["seed"], c["n_pairs"])
    check_parity(q, k, v, lambda0=c["lambda0"], mode=TP, segments=8)


def test_result_is_deterministic():
    """Every reduction has a fixed order (Gram partials summed in wave order, no floating-point atomics): two
    calls on the same inputs agree bit for bit, for the per-wave and for the shared-operand S kernels."""
    import torch

    import paper_2605_11196_amd as vla

    dev = torch.device("cuda:0")
    for heads, T, seg in ((3, 777, 5), (64, 333, 4)):
        q, k, v = (torch.from_numpy(x).to(dev) for x in vla_inputs.gaussian_qkv(1, heads, T, 64, seed=T))
        a = vla.vla_forward(q, k, v, mode=TP, segments=seg)
        b = vla.vla_forward(q, k, v, mode=TP, segments=seg)
        torch.cuda.synchronize()
        for x, y in zip(a, b):
            assert torch.equal(x, y)


def test_segment_count_only_changes_rounding():
    d, T = 64, 1536
    q, k, v = vla_inputs.gaussian_qkv(1, 2, T, d, seed=31)
    ref = gpu_forward(q, k, v, mode=3)
    for segments in (2, 3, 16, 96):
        got = gpu_forward(q, k, v, mode=TP, segments=segments)
        for x, y, nd in zip(got, ref, (2, 2, 2)):
            assert slab_rel_err(x, y, nd) <= 2e-5, segments


@pytest.mark.parametrize("heads", [3, 64])
def test_state_outputs_may_alias_inputs_or_be_null(heads):
    """S_T / A_T written over S0 / A0 (the boundary kernels have read them by then) and left out altogether;
    few heads take the per-wave S kernels, 64 heads x 4 segments the shared-operand ones."""
    import torch

    import paper_2605_11196_amd as vla

    d, T, seg = 64, 200, 4
    dev = torch.device("cuda:0")
    q, k, v = (torch.from_numpy(x).to(dev) for x in vla_inputs.gaussian_qkv(1, heads, T, d, seed=400))
    S0 = torch.randn((1, heads, d, d), device=dev)
    A0 = torch.eye(d, device=dev).expand(1, heads, d, d).contiguous() * 2.0
    o_ref, S_ref, A_ref = vla.vla_forward(q, k, v, S0, A0, mode=TP, segments=seg)
    S_al, A_al = S0.clone(), A0.clone()
    o = torch.empty_like(q)
    need = vla.vla_forward_workspace_bytes(1, heads, T, d, d, vla.VLA_F32, mode=TP, segments=seg)
    ws = torch.empty(need, dtype=torch.uint8, device=dev)
    st = torch.cuda.current_stream().cuda_stream
    args = (1, heads, T, d, d, vla.VLA_F32)
    kw = dict(mode=TP, segments=seg, workspace=ws.data_ptr(), workspace_bytes=need, stream=st)
    rc = vla.vla_forward_raw(q.data_ptr(), k.data_ptr(), v.data_ptr(), S_al.data_ptr(), A_al.data_ptr(),
                             o.data_ptr(), S_al.data_ptr(), A_al.data_ptr(), *args, **kw)
    assert rc == 0
    o2 = torch.empty_like(q)
    rc = vla.vla_forward_raw(q.data_ptr(), k.data_ptr(), v.data_ptr(), S0.data_ptr(), A0.data_ptr(),
                             o2.data_ptr(), 0, 0, *args, **kw)
    assert rc == 0
    torch.cuda.synchronize()
    assert torch.equal(o, o_ref) and torch.equal(S_al, S_ref) and torch.equal(A_al, A_ref)
    assert torch.equal(o2, o_ref)
    ref = oracle.forward(q.cpu().numpy(), k.cpu().numpy(), v.cpu().numpy(), S0.cpu().numpy(), A0.cpu().numpy())
    assert slab_rel_err(o.cpu().numpy(), ref["o"], 2) <= TOL["f32"]
    assert slab_rel_err(S_al.cpu().numpy(), ref["S_T"], 2) <= TOL["f32"]
    assert slab_rel_err(A_al.cpu().numpy(), ref["A_T"], 2) <= TOL["f32"]


def test_workspace_and_option_checks():
    import torch

    import paper_2605_11196_amd as vla

    B, H, T, d = 1, 2, 2048, 64
    need_tp = vla.vla_forward_workspace_bytes(B, H, T, d, d, vla.VLA_F32, mode=TP, segments=4)
    need_2p = vla.vla_forward_workspace_bytes(B, H, T, d, d, vla.VLA_F32, mode=vla.MODE_TWO_PHASE)
    assert need_tp > need_2p > 0
    # AUTO for few heads and a long sequence is this mode and asks for its workspace
    assert vla.resolve_mode(B, H, T, d, d, vla.VLA_F32) == TP
    assert vla.vla_forward_workspace_bytes(B, H, T, d, d, vla.VLA_F32) >= need_2p
    dev = torch.device("cuda:0")
    q = torch.randn(B, H, T, d, device=dev)
    o = torch.empty_like(q)
    ws = torch.empty(need_tp, dtype=torch.uint8, device=dev)
    args = (q.data_ptr(), q.data_ptr(), q.data_ptr(), 0, 0, o.data_ptr(), 0, 0, B, H, T, d, d, vla.VLA_F32)
    # too small a workspace for an explicitly requested mode is an error, nothing is launched
    rc = vla.vla_forward_raw(*args, mode=TP, segments=4, workspace=ws.data_ptr(), workspace_bytes=need_tp - 16)
    assert vla.status_string(rc) == "VLA_ERR_WORKSPACE"
    rc = vla.vla_forward_raw(*args, mode=TP, segments=4, workspace=ws.data_ptr(), workspace_bytes=need_tp)
    assert rc == 0
    # the options of Algorithm 1 break A_t = M_t^{-1} (refresh) or u = k^: refused
    rc = vla.vla_forward_raw(*args, mode=TP, segments=4, workspace=ws.data_ptr(), workspace_bytes=need_tp,
                             refresh_period=20)
    assert vla.status_string(rc) == "VLA_ERR_UNSUPPORTED"
    rc = vla.vla_forward_raw(*args, mode=TP, segments=-1, workspace=ws.data_ptr(), workspace_bytes=need_tp)
    assert vla.status_string(rc) == "VLA_ERR_INVALID_ARG"
    torch.cuda.synchronize()


# ------------------------------------------------------------------ value heads of another size than the key heads
SEG_KEY_SIZES = [32, 64, 96, 128]
VALUE_SIZES = [16, 32, 64, 96, 128]
SEG_RECT_PAIRS = [(dk, dv) for dk in SEG_KEY_SIZES for dv in VALUE_SIZES if dk != dv]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("dk,dv", SEG_RECT_PAIRS)
def test_value_heads_of_another_size_run_in_the_segment_modes(dk, dv, dtype):
    """S is d_v x d_k (eq. (s-update), eq. (output)): the A side of the segment modes only sees the keys, the S rows
    kernel shares the d_v / 16 row slabs of S out to its d_k / 16 waves in turn (one to four slots per wave, some
    waves with none), the per-segment maps are P [d_k][d_k] and Q [d_v][d_k].  Four segments of six blocks with a
    ragged last block and a given S0, time-parallel and two-phase."""
    B, H, T = 2, 3, 333
    q, k, v = vla_inputs.gaussian_qkv(B, H, T, dk, seed=1500 + dk + dv, d_v=dv)
    S0 = np.random.default_rng(dk + dv).standard_normal((B, H, dv, dk)).astype(np.float32)
    for mode, segments in ((TP, 4), (3, None)):
        errs, _, _ = check_parity(q, k, v, S0, None, dtype=dtype, lambda0=0.1, mode=mode, segments=segments)
        print(dk, dv, dtype, mode, errs)


@pytest.mark.parametrize("optset", ["normalised read-out", "penalty direction"])
@pytest.mark.parametrize("dk,dv", [(32, 128), (64, 96), (64, 16), (96, 128), (128, 32), (128, 96)])
def test_options_on_value_heads_of_another_size_in_the_time_parallel_mode(dk, dv, optset):
    """The options the segment modes carry (separate penalty directions, normalised read-out with a carried key
    sum, ELU+1) with d_k != d_v: the A chain of the option kernel feeds the same S rows kernel."""
    import torch

    import paper_2605_11196_amd as vla
    from parity_utils import to_np

    B, H, T = 1, 5, 300
    rng = np.random.default_rng(70 + dk + dv)
    q, k, u = (rng.standard_normal((B, H, T, dk)).astype(np.float32) for _ in range(3))
    v = rng.standard_normal((B, H, T, dv)).astype(np.float32)
    S0 = rng.standard_normal((B, H, dv, dk)).astype(np.float32)
    z0 = np.abs(rng.standard_normal((B, H, dk))).astype(np.float32)
    with_u = optset == "penalty direction"
    opt = dict(lambda0=0.1)
    if with_u:
        opt["u_scale"] = dk ** -0.5
    else:
        opt.update(normalise_output=True, feature_map=True)
    norm = bool(opt.get("normalise_output"))
    ref = oracle.forward(q, k, v, S0, None, u=u if with_u else None, zkey0=z0 if norm else None, **opt)
    dev = torch.device("cuda:0")
    t = lambda x: torch.from_numpy(x).to(dev)
    out = vla.vla_forward(t(q), t(k), t(v), t(S0), None, u=t(u) if with_u else None,
                          zkey0=t(z0) if norm else None, return_zkey=norm, mode=TP, segments=3, **opt)
    torch.cuda.synchronize()
    o, S_T, A_T = out[:3]
    errs = dict(o=slab_rel_err(to_np(o), ref["o"], 2), S=slab_rel_err(to_np(S_T), ref["S_T"], 2),
                A=slab_rel_err(to_np(A_T), ref["A_T"], 2))
    if norm:
        errs["z"] = slab_rel_err(to_np(out[3]), ref["zkey_T"], 1)
    print(dk, dv, optset, errs)
    assert max(errs.values()) <= 1e-4, errs


@pytest.mark.parametrize("dtype,feature_map", [("f32", False), ("bf16", False), ("bf16", True)])
@pytest.mark.parametrize("d,d_v,heads,segments", [
    (128, 128, 32, 8), (128, 64, 32, 8), (128, 128, 86, 3),     # 256 and 258 (head, segment) pairs
    (64, 64, 128, 6), (64, 64, 110, 7), (32, 32, 110, 7),       # 768 and 770
    (64, 128, 40, 4), (96, 64, 40, 4),
])
def test_split_and_fp32_products_on_both_sides_of_their_pair_counts(d, d_v, heads, segments, dtype, feature_map):
    """The pair counts where the S rows and the A scan change kernels, with and without the feature map (one- or
    three-term operands): a one-token last block, a state over eight orders of magnitude, keys of unequal norms."""
    import torch

    import paper_2605_11196_amd as vla

    rng = np.random.default_rng(d + heads + segments)
    T = 16 * segments * 2 - 15
    q, k = (rng.standard_normal((1, heads, T, d)).astype(np.float32) for _ in range(2))
    v = rng.standard_normal((1, heads, T, d_v)).astype(np.float32)
    k *= np.float32(4.0) ** rng.integers(-3, 1 if feature_map else 4, size=(1, heads, T, 1)).astype(np.float32)
    v *= np.float32(10.0) ** rng.integers(-4, 5, size=(1, heads, 1, 1)).astype(np.float32)
    S0 = rng.standard_normal((1, heads, d_v, d)).astype(np.float32) * np.abs(v).max(axis=(2, 3), keepdims=True)
    if dtype == "bf16":
        q, k, v = (vla_inputs.round_to_bf16(x) for x in (q, k, v))
    ref = oracle.forward(q, k, v, S0, None, lambda0=0.1, feature_map=feature_map)
    io = torch.float32 if dtype == "f32" else torch.bfloat16
    tq, tk, tv = (torch.from_numpy(x).cuda().to(io) for x in (q, k, v))
    got = vla.vla_forward(tq, tk, tv, torch.from_numpy(S0).cuda(), None, lambda0=0.1, feature_map=feature_map, mode=TP,
                          segments=segments)
    for name, x in zip(("o", "S_T", "A_T"), got):
        err = slab_rel_err(x.float().cpu().numpy(), ref[name], 2)
        print(d, d_v, heads, segments, dtype, feature_map, name, err)
        assert err <= TOL[dtype], (name, err)


@pytest.mark.parametrize("given", [False, True])
@pytest.mark.parametrize("segments", [2, 5, 6, 7])
@pytest.mark.parametrize("d", [32, 64, 96, 128])
def test_gram_matrices_added_up_in_front_of_the_inverse_or_by_a_kernel(d, segments, given):
    """Six segments are the last whose sums the boundary inverse forms itself, two at a time: odd and even counts and the first
    count that has them summed before, from an identity and from a given A0."""
    q, k, v = vla_inputs.gaussian_qkv(2, 2, 32 * segments - 3, d, seed=1900 + segments)
    A0 = None
    if given:
        m = np.random.default_rng(d).standard_normal((2, 2, d, d)).astype(np.float32) / np.sqrt(d)
        A0 = np.eye(d, dtype=np.float32) + m @ m.transpose(0, 1, 3, 2)
        A0 = (0.5 * (A0 + A0.transpose(0, 1, 3, 2))).astype(np.float32)
    check_parity(q, k, v, None, A0, dtype="f32", lambda0=0.1, mode=TP, segments=segments)


@pytest.mark.parametrize("dtype,feature_map", [("f32", False), ("bf16", False), ("bf16", True)])
@pytest.mark.parametrize("d,d_v", [(32, 16), (32, 64), (32, 96), (32, 128), (64, 64), (64, 96), (96, 96), (96, 128), (128, 16), (128, 128)])
def test_maps_beside_the_a_chain_in_every_slot_layout(d, d_v, dtype, feature_map):
    """Segments of one block, of one token more and of several blocks; every number of row slabs per map wave and both
    numbers of operand terms; given states."""
    rng = np.random.default_rng(d * d_v)
    for T, segments in ((33, 3), (17, 2), (150, 3)):
        q, k, _ = vla_inputs.gaussian_qkv(2, 2, T, d, seed=T)
        v = rng.standard_normal((2, 2, T, d_v)).astype(np.float32)
        S0 = rng.standard_normal((2, 2, d_v, d)).astype(np.float32)
        m = rng.standard_normal((2, 2, d, d)).astype(np.float32) / np.sqrt(d)
        A0 = np.eye(d, dtype=np.float32) + m @ m.transpose(0, 1, 3, 2)
        A0 = (0.5 * (A0 + A0.transpose(0, 1, 3, 2))).astype(np.float32)
        check_parity(q, k, v, S0, A0, dtype=dtype, mode=TP, segments=segments, feature_map=feature_map)


@pytest.mark.parametrize("dtype,feature_map", [("f32", False), ("bf16", False), ("bf16", True)])
@pytest.mark.parametrize("heads", [128, 129])
def test_maps_of_five_slots_in_up_to_one_workgroup_a_compute_unit_and_in_more(heads, dtype, feature_map):
    """Two segments of a head: 256 pairs and the first count above."""
    q, k, _ = vla_inputs.gaussian_qkv(1, heads, 53, 32, seed=heads)
    v = np.random.default_rng(heads).standard_normal((1, heads, 53, 128)).astype(np.float32)
    check_parity(q, k, v, None, None, dtype=dtype, mode=TP, segments=2, feature_map=feature_map)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d,T,segments,lambda0", [
    (32, 16 * 9 + 5, 3, 0.1), (64, 16 * 12 + 1, 3, 0.1), (96, 16 * 8 + 15, 2, 0.1), (128, 16 * 9, 3, 0.1),   # ragged tiles of 64 and 128 tokens
    (32, 40000, 2, 0.1),            # more tokens in a segment than one set of integer sums takes
    (64, 900, 4, 0.01), (64, 900, 4, 0.009),   # both sides of the smallest lambda0 in fixed point
])
# (no larger scale: A goes from 10 to lambda0 / u_scale^2 within d tokens, and the first segment's float32 recurrence loses as much,
# in float64 sums and in these alike: heads of 32, 30: 8e-4 of o, 300: 3e-2)
@pytest.mark.parametrize("u_scale", [None, 0.3, 3.0, 1e-3])
def test_fixed_point_gram_sums(d, T, segments, lambda0, u_scale, dtype):
    """A after the last segment starts from the inverse of the summed directions: against the oracle, with and without given
    directions whose scale is no power of two, large or small.  Bound of A: four times what is measured (1.2e-6; 2.6e-6 after
    20000 float32 steps), which float64 sums show alike; S: that of the I/O type, as everywhere."""
    import torch

    import paper_2605_11196_amd as vla

    rng = np.random.default_rng(T)
    heads = 1 if T > 10000 else 3
    q, k, v = vla_inputs.gaussian_qkv(1, heads, T, d, seed=T + d)
    u = rng.standard_normal(k.shape).astype(np.float32) if u_scale is not None else None
    if dtype == "bf16":
        q, k, v = (vla_inputs.round_to_bf16(x) for x in (q, k, v))
        u = None if u is None else vla_inputs.round_to_bf16(u)
    opt = dict(lambda0=lambda0) if u is None else dict(lambda0=lambda0, u_scale=u_scale)
    ref = oracle.forward(q, k, v, u=u, **opt)
    t = lambda x: None if x is None else torch.from_numpy(x).cuda().to(torch.float32 if dtype == "f32" else torch.bfloat16)
    _, S_T, A_T = vla.vla_forward(t(q), t(k), t(v), u=t(u), mode=TP, segments=segments, **opt)
    torch.cuda.synchronize()
    err = slab_rel_err(A_T.cpu().numpy(), ref["A_T"], 2)
    print(d, T, segments, lambda0, u_scale, dtype, err)
    assert err <= (1e-5 if T > 10000 else 5e-6)
    assert slab_rel_err(S_T.cpu().numpy(), ref["S_T"], 2) <= 1e-4


@pytest.mark.parametrize("d,T,lambda0,distinct", [(32, 100000, 0.1, 1), (64, 100000, 0.1, 1), (64, 100000, 0.1, 4), (96, 50000, 0.1, 1),
                                                  (128, 100000, 0.1, 1), (64, 20000, 0.01, 1), (64, 100000, 0.01, 1)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_keys_seen_over_and_over_leave_a_alone_elsewhere(d, T, lambda0, distinct, dtype):
    """What a sum of equal products leaves out adds up, and off the keys A is 1 / lambda0 and nothing else.  A from its definition
    in float64.  The float32 steps of the last segment lose up to 3e-7 of A with fixed-point and with float64 sums, 2.6e-6
    where one key stands 1e7 times above lambda0 (float64 sums)."""
    import torch

    import paper_2605_11196_amd as vla

    rng = np.random.default_rng(d + T)
    k = rng.standard_normal((distinct, d)).astype(np.float32)
    k = vla_inputs.round_to_bf16(k) if dtype == "bf16" else k
    kn = k.astype(np.float64) / np.linalg.norm(k.astype(np.float64), axis=1, keepdims=True)
    ref = np.linalg.inv(np.float64(np.float32(lambda0)) * np.eye(d) + (T // distinct) * kn.T @ kn)
    dev = torch.device("cuda:0")
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    tk = torch.from_numpy(k).to(dev).to(tdt).repeat(T // distinct, 1)[None, None]
    q, v = (torch.randn((1, 1, T, d), device=dev, dtype=tdt) for _ in range(2))
    _, _, A_T = vla.vla_forward(q, tk, v, lambda0=lambda0, mode=TP)
    torch.cuda.synchronize()
    err = np.abs(A_T[0, 0].cpu().numpy() - ref).max() / np.abs(ref).max()
    print(d, T, lambda0, distinct, dtype, err)
    assert err <= (1e-6 if T / distinct <= 2e6 * lambda0 else 1e-5)


@pytest.mark.parametrize("u_scale", [1.0, -1.0, 100.0, 1000.0, 30000.0])
@pytest.mark.parametrize("d", [32, 64, 128])
def test_short_directions_of_a_large_scale(d, u_scale):
    """One direction far below eps, whose sum over the tokens is as large as lambda0, against A from its definition in
    float64.  2e-6: the float32 norm of the direction counts twice, and 4096 float32 steps of the last segment."""
    import torch

    import paper_2605_11196_amd as vla

    T, lambda0, eps = 65536, 0.01, 1e-4
    rng = np.random.default_rng(d)
    x = rng.standard_normal(d)
    u = (x / np.linalg.norm(x) * eps * np.sqrt(lambda0 / T) / abs(u_scale)).astype(np.float32)
    un = np.float64(np.float32(u_scale)) * u.astype(np.float64) / np.float64(np.float32(eps))
    ref = np.linalg.inv(np.float64(np.float32(lambda0)) * np.eye(d) + T * np.outer(un, un))
    dev = torch.device("cuda:0")
    tu = torch.from_numpy(u).to(dev).repeat(T, 1)[None, None]
    q, k, v = (torch.randn((1, 1, T, d), device=dev) for _ in range(3))
    _, _, A_T = vla.vla_forward(q, k, v, lambda0=lambda0, eps=eps, u=tu, u_scale=u_scale, mode=TP)
    torch.cuda.synchronize()
    err = np.abs(A_T[0, 0].cpu().numpy() - ref).max() / np.abs(ref).max()
    print(d, u_scale, err)
    assert err <= 2e-6


@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("d", [32, 64, 96, 128])
def test_a_key_that_is_not_finite_reaches_every_later_segment_of_its_head_only(d, value):
    import torch

    import paper_2605_11196_amd as vla

    q, k, v = (torch.from_numpy(x).cuda() for x in vla_inputs.gaussian_qkv(1, 2, 200, d, seed=d))
    k[0, 1, 20, 3] = value
    o, S_T, A_T = vla.vla_forward(q, k, v, lambda0=0.1, mode=TP, segments=4)
    torch.cuda.synchronize()
    assert torch.isfinite(o[0, 0]).all() and torch.isfinite(A_T[0, 0]).all()
    assert torch.isnan(A_T[0, 1]).any() and torch.isnan(o[0, 1, 64:]).any(dim=-1).all()
