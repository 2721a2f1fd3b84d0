"""GPU parity of the prefill path (App. A.5) against the oracle: a chunk of T
tokens per request runs in fp32 from the decoded stored state, o for every
token, and only the chunk-final state is stored. Both sides start from
identical bytes packed by the oracle (see parity_util for the bar).
"""
import numpy as np
import pytest
import torch

from oracle import oracle as orc
from paper_2608_27513_amd import damp as D
from paper_2608_27513_amd import inputs
from parity_util import O_TOL_MIXED, compare_tiles, dev_i32, dev_inputs, dev_u8, gpu_pool_from, rel_l2

pytestmark = pytest.mark.gpu


def _say(*a):
    print(*a, flush=True)


def _run(kda, ref, gpool, slots, inp, perm, scale=1.0, o_dtype=torch.float32):
    d_inp = dev_inputs(inp)
    B, T = inp["q"].shape[:2]
    o = torch.empty((B, T, ref.hv, ref.dv), dtype=o_dtype, device="cuda")
    fn = D.damp_state_prefill_kda if kda else D.damp_state_prefill_gdn
    fn(gpool, 0, dev_i32(slots), d_inp["q"], d_inp["k"], d_inp["v"], d_inp["g"], d_inp["beta"],
       perm=None if perm is None else dev_u8(perm), scale=scale, o=o)
    o_ref = orc.prefill(ref, 0, slots, kda=kda, perm=perm, scale=scale, **inp)
    torch.cuda.synchronize()
    return o.float().cpu().numpy(), o_ref


CASES = [
    # (d, kda, HK, HV, B, T, k_hi, kind, fmt)
    (16, False, 1, 2, 2, 5, 4, orc.KIND_MIXED, None),
    (16, True, 2, 2, 2, 3, 0, orc.KIND_FP32, None),
    (32, False, 2, 4, 3, 8, 8, orc.KIND_MIXED, None),
    (32, True, 2, 2, 2, 4, 8, orc.KIND_MIXED, orc.FMT_PAPER),
    (64, True, 4, 4, 2, 16, 16, orc.KIND_MIXED, None),
    (64, False, 2, 4, 2, 6, 0, orc.KIND_FP32, None),
    (128, False, 2, 4, 2, 16, 16, orc.KIND_MIXED, None),
    (128, True, 4, 4, 2, 8, 16, orc.KIND_MIXED, None),
    (128, False, 2, 4, 2, 8, 16, orc.KIND_MIXED, orc.FMT_PAPER),
    (128, True, 2, 2, 2, 1, 32, orc.KIND_MIXED, None),
    (128, False, 2, 2, 2, 12, 0, orc.KIND_FP32, None),
    # d = 128 runs in chunks of 16 tokens: one token past a chunk; several
    # chunks, with decays whose product vanishes; the other formats
    (128, True, 2, 2, 2, 17, 12, orc.KIND_MIXED, None),
    (128, False, 2, 2, 2, 48, 16, orc.KIND_MIXED, None),
    (128, False, 2, 4, 3, 24, 16, orc.KIND_MIXED, orc.FMT_INT4_H32),
    (128, True, 2, 2, 2, 9, 16, orc.KIND_MIXED, orc.FMT_FP8),
    (128, False, 2, 2, 2, 11, 16, orc.KIND_MIXED, orc.FMT_NVFP4),
]


@pytest.mark.parametrize("d,kda,HK,HV,B,T,k_hi,kind,fmt", CASES)
def test_prefill_parity(d, kda, HK, HV, B, T, k_hi, kind, fmt):
    _say(f"prefill d={d} kda={kda} HK={HK} HV={HV} B={B} T={T} k_hi={k_hi} kind={kind} fmt={fmt}")
    seed = 700 + d + T + k_hi + 5 * kda + (fmt is not None)
    slots = inputs.slot_order(seed, B + 2, B)
    perm = inputs.random_perms(seed, HV, d)
    S = inputs.synthetic_states(seed, B, HV, d)
    ref = orc.Pool(kind, d, d, k_hi, 1, B + 2, HV, fmt=fmt)
    orc.pack(ref, 0, slots, S, perm)
    gpool = gpu_pool_from(ref, D)
    inp = inputs.as_prefill(inputs.decode_inputs(seed, T, B, HK, HV, d, kda=kda))
    o_gpu, o_ref = _run(kda, ref, gpool, slots, inp, perm, scale=0.75)
    err = rel_l2(o_gpu, o_ref)
    # T fp32 steps before the one FP16 rounding of the scales: a scale within
    # one FP16 step everywhere, equal on 99% (codes keep the 99.9% bar)
    stats = compare_tiles(gpool.buffer.cpu().numpy(), ref, f"prefill d={d}", s16_exact_min=0.99)
    _say(f"  o rel-L2 {err:.2e}  {stats}")
    if kind == orc.KIND_FP32:
        assert err <= 1e-5
    else:
        assert err <= O_TOL_MIXED
        assert err <= 1e-4  # identical starting bytes, no quantization inside the chunk


@pytest.mark.parametrize("d,T", [(64, 4), (128, 10)])
def test_prefill_padded_requests_and_bf16_output(d, T):
    HK, HV, B = 2, 4, 3
    ref = orc.Pool(orc.KIND_MIXED, d, d, 8, 1, 4, HV)
    orc.pack(ref, 0, np.arange(4), inputs.synthetic_states(710, 4, HV, d))
    pad = 4096
    raw = torch.full((ref.buf.size + 2 * pad,), 0xA5, dtype=torch.uint8, device="cuda")
    raw[pad:pad + ref.buf.size] = torch.from_numpy(ref.buf).cuda()
    gpool = D.Pool(D.damp_layout_init(d, d, 8), 1, 4, HV, buffer=raw[pad:pad + ref.buf.size])
    slots = np.array([2, -1, 4], np.int32)  # -1 padded, 4 == num_slots out of range
    inp = inputs.as_prefill(inputs.decode_inputs(711, T, B, HK, HV, d))
    o_gpu, o_ref = _run(False, ref, gpool, slots, inp, None, o_dtype=torch.bfloat16)
    assert (o_gpu[1] == 0).all() and (o_gpu[2] == 0).all()
    assert rel_l2(o_gpu, o_ref) <= 4e-3  # bf16 rounding of o
    host = raw.cpu().numpy()
    assert (host[:pad] == 0xA5).all() and (host[-pad:] == 0xA5).all()
    compare_tiles(host[pad:-pad], ref, "prefill padded")
    st = ref.slot_stride
    for s in (0, 1, 3):
        assert np.array_equal(host[pad + s * st:pad + (s + 1) * st], ref.buf[s * st:(s + 1) * st])


def test_prefill_kda_blocks_with_vanishing_decay():
    """KDA at d = 128 refers a chunk of 16 tokens to its middle token unless a
    channel's product on either side of it leaves [2^-80, 2^80]; here the
    second of four chunks holds a channel decaying by e^-12 per token (product
    e^-96 over eight) and one token with a zero decay (g = -inf), between
    chunks without such channels."""
    d, HK, HV, B, T, k_hi = 128, 2, 2, 2, 56, 16
    seed = 733
    slots = inputs.slot_order(seed, B + 2, B)
    perm = inputs.random_perms(seed, HV, d)
    ref = orc.Pool(orc.KIND_MIXED, d, d, k_hi, 1, B + 2, HV)
    orc.pack(ref, 0, slots, inputs.synthetic_states(seed, B, HV, d), perm)
    gpool = gpu_pool_from(ref, D)
    inp = inputs.as_prefill(inputs.decode_inputs(seed, T, B, HK, HV, d, kda=True))
    g = inp["g"].copy()  # bf16 bits [B, T, HV, d]
    g[0, 24:32, 0, 5] = inputs.to_bf16_bits(np.float32(-12.0))[0]
    g[1, 28, 1, 70] = inputs.to_bf16_bits(np.float32(-np.inf))[0]
    inp["g"] = g
    o_gpu, o_ref = _run(True, ref, gpool, slots, inp, perm)
    err = rel_l2(o_gpu, o_ref)
    stats = compare_tiles(gpool.buffer.cpu().numpy(), ref, "prefill KDA vanishing decay",
                          s16_exact_min=0.99)
    _say(f"  o rel-L2 {err:.2e}  {stats}")
    assert err <= 1e-4


def test_prefill_gdn_vanishing_and_zero_decay():
    """GDN at d = 128 takes the decays of a chunk of 16 tokens as running
    products, which may vanish. Here, in the second of four chunks: a zero
    decay (g = -inf), decays below the smallest normal fp32 number (g = -100,
    -90), and a run of e^-5 decays; and a zero decay at the first token of the
    third."""
    d, HK, HV, B, T, k_hi = 128, 1, 2, 2, 56, 16
    seed = 741
    slots = inputs.slot_order(seed, B + 2, B)
    perm = inputs.random_perms(seed, HV, d)
    ref = orc.Pool(orc.KIND_MIXED, d, d, k_hi, 1, B + 2, HV)
    orc.pack(ref, 0, slots, inputs.synthetic_states(seed, B, HV, d), perm)
    gpool = gpu_pool_from(ref, D)
    inp = inputs.as_prefill(inputs.decode_inputs(seed, T, B, HK, HV, d))
    g = inp["g"].copy()  # bf16 bits [B, T, HV]
    bits = lambda x: inputs.to_bf16_bits(np.float32(x))[0]
    g[0, 19, 0] = bits(-np.inf)
    g[0, 26, 0] = bits(-100.0)
    g[1, 18:28, 1] = bits(-5.0)
    g[1, 30, 1] = bits(-90.0)
    g[0, 32, 1] = bits(-np.inf)
    inp["g"] = g
    o_gpu, o_ref = _run(False, ref, gpool, slots, inp, perm)
    assert np.isfinite(o_gpu).all()
    err = rel_l2(o_gpu, o_ref)
    stats = compare_tiles(gpool.buffer.cpu().numpy(), ref, "prefill GDN vanishing decay",
                          s16_exact_min=0.99)
    _say(f"  o rel-L2 {err:.2e}  {stats}")
    assert err <= 1e-4


def test_calibrate_sequence_gdn_vanishing_decay():
    """The calibration trajectory of GDN at d = 128 runs through the same
    chunked prefill kernel, a window of one stride at a time: zero and sub-normal decays (g = -inf,
    -100) between the sampled tokens keep the FP32 trajectory finite and
    equal to the oracle's."""
    d, H, HK, B, T = 128, 2, 1, 2, 24
    inp = inputs.decode_inputs(743, T, B, HK, H, d)
    bits = lambda x: inputs.to_bf16_bits(np.float32(x))[0]
    g = inp["g"].copy()  # step-major [T, B, H]
    g[3, 0, 0] = bits(-np.inf)
    g[10, 1, 1] = bits(-100.0)
    g[12:14, 0, 1] = bits(-60.0)
    inp["g"] = g
    cal_ref = orc.Calib(kda=False, H=H, dk=d, dv=d)
    S_ref = orc.calibrate_sequence(cal_ref, 0, np.zeros((B, H, d, d), np.float32), stride=8, **inp)
    pool = D.Pool(D.damp_layout_init(d, d, 0, D.DAMP_STATE_FP32), 1, B, H)
    slots = torch.arange(B, dtype=torch.int32, device="cuda")
    D.damp_pool_reset_slots(pool, 0, slots)
    cal = D.Calib(D.damp_layout_init(d, d, 0), kda=False, num_heads=H)
    x = {n: torch.from_numpy(np.ascontiguousarray(np.swapaxes(a, 0, 1)).view(np.int16)).cuda()
         .view(torch.bfloat16) for n, a in inp.items()}
    D.damp_calibrate_sequence(cal, 0, pool, 0, slots, x["q"], x["k"], x["v"], x["g"], x["beta"])
    S_gpu = D.damp_state_unpack(pool, 0, slots).cpu().numpy()
    torch.cuda.synchronize()
    assert np.isfinite(S_gpu).all()
    assert np.linalg.norm(S_gpu - S_ref) <= 1e-5 * np.linalg.norm(S_ref)
    h = cal.buffer.cpu().numpy()
    sums = h[:3 * H * d].reshape(3, H, d)
    assert np.isfinite(sums).all()
    np.testing.assert_allclose(sums[0], cal_ref.sums[0, 0], rtol=2e-3)
    np.testing.assert_allclose(sums[1], cal_ref.sums[0, 1], rtol=1e-5)


@pytest.mark.parametrize("B", [2, 129])
@pytest.mark.parametrize("kda", [False, True])
@pytest.mark.parametrize("T", [1, 4, 5, 15, 16, 17, 33, 64, 65, 130])
def test_prefill_chunk_edges(kda, T, B):
    """d = 128 runs in chunks of 16 tokens, several staged together: one token,
    the edges of the four-row groups, of a chunk and of a staging block, and a
    partial last chunk; with up to 256 tiles staged by waves of their own, with
    more (B = 129, two heads) by the waves that run them. FP32 state, so o and
    the state carry fp32 rounding only: 7e-8 to 3.4e-7 measured, and 2.2e-6 to
    1.1e-5 with the third part of the state's splits left out, so a bar of 1e-6
    pins that part."""
    d, HK, HV = 128, 2 if kda else 1, 2
    seed = 760 + T
    slots = inputs.slot_order(seed, B + 1, B)
    perm = inputs.random_perms(seed, HV, d)
    ref = orc.Pool(orc.KIND_FP32, d, d, 0, 1, B + 1, HV)
    orc.pack(ref, 0, slots, inputs.synthetic_states(seed, B, HV, d), perm)
    gpool = gpu_pool_from(ref, D)
    inp = inputs.as_prefill(inputs.decode_inputs(seed, T, B, HK, HV, d, kda=kda))
    o_gpu, o_ref = _run(kda, ref, gpool, slots, inp, perm)
    state = gpool.buffer.cpu().numpy().view(np.float32)
    err, s_err = rel_l2(o_gpu, o_ref), rel_l2(state, ref.buf.view(np.float32))
    _say(f"  T={T} kda={kda} o rel-L2 {err:.2e} state rel-L2 {s_err:.2e}")
    assert err <= 1e-6 and s_err <= 1e-6


@pytest.mark.parametrize("kda", [False, True])
@pytest.mark.parametrize("B", [2, 129])
def test_prefill_inputs_at_odd_addresses(kda, B):
    """q, k, v and g 2 or 4 bytes off: the d = 128 kernel reads k, q and KDA's
    g by halves where they are not word aligned, and 16 bytes at a time where
    they are: the same outputs and state."""
    d, HK, HV, T = 128, 2, 2, 21
    seed = 790
    ref = orc.Pool(orc.KIND_FP32, d, d, 0, 1, B, HV)
    orc.pack(ref, 0, np.arange(B), inputs.synthetic_states(seed, B, HV, d))
    inp = dev_inputs(inputs.as_prefill(inputs.decode_inputs(seed, T, B, HK, HV, d, kda=kda)))
    fn = D.damp_state_prefill_kda if kda else D.damp_state_prefill_gdn

    def shifted(t, by):  # the same values, 2 by bytes off
        raw = torch.empty(t.numel() + by, dtype=t.dtype, device="cuda")
        raw[by:] = t.reshape(-1)
        return raw[by:].view(t.shape)

    got = []
    for odd, by in (((), 0), (("q",), 1), (("k",), 1), (("v",), 1), (("g",), 1),
                    (("q", "k", "v", "g", "beta"), 1), (("q", "k", "v", "g", "beta"), 2)):
        pool = gpu_pool_from(ref, D)
        a = {n: shifted(t, by) if n in odd else t for n, t in inp.items()}
        o = fn(pool, 0, dev_i32(np.arange(B)), a["q"], a["k"], a["v"], a["g"], a["beta"])
        got.append((o.cpu().numpy(), pool.buffer.cpu().numpy().view(np.float32)))
    for o, s in got[1:]:
        assert np.array_equal(o, got[0][0]) and np.array_equal(s, got[0][1])


@pytest.mark.parametrize("kda", [False, True])
@pytest.mark.parametrize("B", [1, 258])
@pytest.mark.parametrize("what", ["v", "k", "q"])
def test_prefill_nonfinite_input_leaves_earlier_tokens(kda, what, B):
    """An infinite input value at one token: every earlier token's output, and
    for v and q everything the recurrence does not reach (other columns;
    later tokens and the state), is what it is without it."""
    d, HK, HV, T, at = 128, 1, 1, 40, 21
    seed = 795
    ref = orc.Pool(orc.KIND_FP32, d, d, 0, 1, B, HV)
    orc.pack(ref, 0, np.arange(B), inputs.synthetic_states(seed, B, HV, d))
    inp = inputs.as_prefill(inputs.decode_inputs(seed, T, B, HK, HV, d, kda=kda))
    fn = D.damp_state_prefill_kda if kda else D.damp_state_prefill_gdn
    res = []  # of request 0
    for bad in (False, True):
        x = {n: a.copy() for n, a in inp.items()}
        if bad:
            x[what][0, at, 0, 37] = 0x7f80  # +inf
        pool = gpu_pool_from(ref, D)
        a = dev_inputs(x)
        o = fn(pool, 0, dev_i32(np.arange(B)), a["q"], a["k"], a["v"], a["g"], a["beta"])
        res.append((o[0, :, 0].cpu().numpy(),
                    pool.buffer.cpu().numpy().view(np.float32).reshape(-1)[:d * d].reshape(d, d)))
    (o0, s0), (o1, s1) = res
    assert rel_l2(o1[:at], o0[:at]) <= 1e-5
    assert not np.isfinite(o1[at]).all()
    if what == "v":  # its column from there on, no other
        keep = np.arange(d) != 37
        assert rel_l2(o1[:, keep], o0[:, keep]) <= 1e-5
        assert rel_l2(s1[:, keep], s0[:, keep]) <= 1e-5
        assert not np.isfinite(s1[:, 37]).any()
    if what == "q":
        keep = np.arange(T) != at
        assert rel_l2(o1[keep], o0[keep]) <= 1e-5 and rel_l2(s1, s0) <= 1e-5


@pytest.mark.parametrize("kda", [False, True])
def test_prefill_vanishing_decays_with_many_tiles(kda):
    """Zero decays and decays whose products leave the range of the chunk form,
    in a batch of more than 256 tiles, every request against the oracle."""
    d, HK, HV, B, T = 128, 1, 1, 260, 50
    seed = 797
    ref = orc.Pool(orc.KIND_FP32, d, d, 0, 1, B, HV)
    orc.pack(ref, 0, np.arange(B), inputs.synthetic_states(seed, B, HV, d))
    gpool = gpu_pool_from(ref, D)
    inp = inputs.as_prefill(inputs.decode_inputs(seed, T, B, HK, HV, d, kda=kda))
    g = inp["g"].copy()
    bits = lambda x: inputs.to_bf16_bits(np.float32(x))[0]
    g[0::3, 20] = bits(-np.inf)
    if kda:
        g[1::3, 17:30, 0, 9] = bits(-20.0)
        g[2::3, 40:, 0, 100] = bits(-90.0)
    else:
        g[1::3, 17:30] = bits(-20.0)
        g[2::3, 40:] = bits(-90.0)
    inp["g"] = g
    o_gpu, o_ref = _run(kda, ref, gpool, np.arange(B), inp, None)
    state = gpool.buffer.cpu().numpy().view(np.float32)
    assert np.isfinite(o_gpu).all() and np.isfinite(state).all()
    assert rel_l2(o_gpu, o_ref) <= 1e-6 and rel_l2(state, ref.buf.view(np.float32)) <= 1e-6


def _fp32_case(kda, B, HV, T, seed, states=None, HK=None):
    """d = 128, FP32 state, identity slots: (oracle pool, GPU pool, inputs)."""
    d, HK = 128, HK or HV
    ref = orc.Pool(orc.KIND_FP32, d, d, 0, 1, B, HV)
    S = np.zeros((B, HV, d, d), np.float32) if states is None else states
    orc.pack(ref, 0, np.arange(B), S)
    return ref, gpu_pool_from(ref, D), inputs.as_prefill(
        inputs.decode_inputs(seed, T, B, HK, HV, d, kda=kda))


def _bits(x):
    return inputs.to_bf16_bits(np.float32(x))[0]


def _scale_bf16(bits, factor):
    """bf16 bit patterns times a power of two (exact)."""
    return inputs.to_bf16_bits((bits.astype(np.uint32) << 16).view(np.float32) * np.float32(factor))


@pytest.mark.parametrize("B", [2, 129])
def test_prefill_gdn_growing_factors(B):
    """Factors above one whose product over a chunk is beyond fp32, on a state
    that is still zero: the state stays zero through them. In head 0 the
    product from the chunk's start overflows, in head 1 only the one from its
    second token on."""
    HV, T = 2, 40
    ref, gpool, inp = _fp32_case(False, B, HV, T, 801)
    g, v = inp["g"].copy(), inp["v"].copy()
    g[:, :12, 0] = _bits(10.0)
    g[:, 0, 1] = _bits(-50.0)
    g[:, 1:10, 1] = _bits(12.0)
    v[:, :12] = 0
    inp.update(g=g, v=v)
    o_gpu, o_ref = _run(False, ref, gpool, np.arange(B), inp, None)
    state = gpool.buffer.cpu().numpy().view(np.float32)
    assert np.isfinite(o_gpu).all() and np.isfinite(state).all()
    assert rel_l2(o_gpu, o_ref) <= 1e-6 and rel_l2(state, ref.buf.view(np.float32)) <= 1e-6


@pytest.mark.parametrize("B", [2, 129])
@pytest.mark.parametrize("kda", [False, True])
def test_prefill_overflow_leaves_earlier_tokens(kda, B):
    """Keys of norm 128: each token multiplies the state by up to |k|^2, which
    leaves fp32 within the first chunk. The tokens before that are what they
    are in the token-by-token form (whose rounding grows with the state: its
    bar is looser here). A single large key in an otherwise ordinary chunk
    overflows one token's read-outs and what follows it, nothing before."""
    HV, T = 1, 16
    S = inputs.synthetic_states(803, B, HV, 128)
    ref, gpool, inp = _fp32_case(kda, B, HV, T, 803, S)
    inp["k"] = _scale_bf16(inp["k"], 128.0)
    o_gpu, o_ref = _run(kda, ref, gpool, np.arange(B), inp, None)
    with np.errstate(all="ignore"):
        top = np.abs(o_ref).max((0, 2, 3))
    fine = np.flatnonzero(~(top < 1e30))
    before = int(fine[0]) if fine.size else T
    assert before < T  # it does overflow
    for t in range(before):
        assert rel_l2(o_gpu[:, t], o_ref[:, t]) <= 1e-4, t

    ref, gpool, inp = _fp32_case(kda, B, HV, T, 805, S * np.float32(2.0 ** 70))
    k = inp["k"].copy()
    k[:, 9] = _scale_bf16(k[:, 9], 2.0 ** 70)
    inp["k"] = k
    o_gpu, o_ref = _run(kda, ref, gpool, np.arange(B), inp, None)
    assert rel_l2(o_gpu[:, :9], o_ref[:, :9]) <= 1e-6
    assert not np.isfinite(o_gpu[:, 10:]).any()


# steep channels: one; a few of both halves of the channels, even and odd; as
# many of one half as are taken at a time, and one more; every channel
STEEP = {"one": [37], "both_waves": [2, 5, 64, 127], "batch": list(range(8, 16)),
         "batch_and_one": list(range(70, 79)), "all": list(range(128))}


@pytest.mark.parametrize("B", [2, 257])
@pytest.mark.parametrize("g0", [-9.5, -30.0, -100.0, -np.inf])
@pytest.mark.parametrize("which", list(STEEP))
def test_prefill_kda_steep_channels(which, g0, B):
    """Channels whose decays over half a chunk leave the range of the matrix
    form, beside ordinary ones: in every token, in the first or the second
    half of a chunk only, at one token inside a half (in a chunk between
    ordinary ones) and in a partial last chunk."""
    HV, T, seed = 1, 74, 811
    S = inputs.synthetic_states(seed, B, HV, 128)
    ref, gpool, inp = _fp32_case(True, B, HV, T, seed, S)
    g = inp["g"].copy()
    for b, span in enumerate((slice(0, T), slice(16, 24), slice(24, 32), slice(20, 21),
                              slice(64, T), slice(39, 41))):
        for c in STEEP[which]:
            g[b::6, span, 0, c] = _bits(g0)
    inp["g"] = g
    o_gpu, o_ref = _run(True, ref, gpool, np.arange(B), inp, None)
    state = gpool.buffer.cpu().numpy().view(np.float32)
    err, s_err = rel_l2(o_gpu, o_ref), rel_l2(state, ref.buf.view(np.float32))
    _say(f"  {which} g={g0} B={B}: o rel-L2 {err:.2e} state rel-L2 {s_err:.2e}")
    assert err <= 1e-6 and s_err <= 1e-6


def test_prefill_kda_steep_channel_costs_little():
    """One channel of 128 that decays steeply leaves the others in the matrix
    form: 1.5 times the time of the batch without it here, 5 times if the
    whole tile ran token by token."""
    HV, B, T = 4, 2, 512
    _, gpool, inp = _fp32_case(True, B, HV, T, 821)
    ms = []
    for steep in (False, True):
        x = dict(inp, g=inp["g"].copy())
        if steep:
            x["g"][..., 7] = _bits(-9.0)
        x, slots = dev_inputs(x), dev_i32(np.arange(B))
        call = lambda: D.damp_state_prefill_kda(gpool, 0, slots, x["q"], x["k"], x["v"], x["g"],
                                                x["beta"])
        call()
        runs = []
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(4):
                call()
            b.record()
            b.synchronize()
            runs.append(a.elapsed_time(b))
        ms.append(min(runs))
    _say(f"  {ms[0] / 4 * 1e3:.1f} us, with a steep channel {ms[1] / 4 * 1e3:.1f} us")
    assert ms[1] <= 3 * ms[0]


@pytest.mark.parametrize("B", [2, 129])
@pytest.mark.parametrize("power", [100, 60, 33, 28, -20, -25, -60, -90])
@pytest.mark.parametrize("kda", [False, True])
def test_prefill_scale_of_state_and_values(kda, power, B):
    """The recurrence is linear in (state, v): their scale costs no precision,
    from where a chunk's products would overflow to where a part of a split
    would fall below the normal numbers. Some of KDA's channels decay by 2^-79
    on either side of a chunk's middle, just inside the range of the matrix
    form."""
    HV, T, seed = 2, 40, 831
    S = inputs.synthetic_states(seed, B, HV, 128) * np.float32(2.0 ** power)
    ref, gpool, inp = _fp32_case(kda, B, HV, T, seed, S)
    inp["v"] = _scale_bf16(inp["v"], 2.0 ** power)
    if kda:
        g = inp["g"].copy()
        g[..., 3::16] = _bits(-79 * np.log(2.0) / 8)
        inp["g"] = g
    o_gpu, o_ref = _run(kda, ref, gpool, np.arange(B), inp, None)
    state = gpool.buffer.cpu().numpy().view(np.float32)
    err, s_err = rel_l2(o_gpu, o_ref), rel_l2(state, ref.buf.view(np.float32))
    _say(f"  kda={kda} 2^{power} B={B}: o rel-L2 {err:.2e} state rel-L2 {s_err:.2e}")
    assert err <= 1e-6 and s_err <= 1e-6


@pytest.mark.parametrize("kda", [False, True])
@pytest.mark.parametrize("kind", ["fp32", "mixed"])
@pytest.mark.parametrize("HV,T", [(131071, 49), (131080, 3)])
def test_prefill_as_many_heads_as_the_chunked_kernel_addresses(HV, T, kind, kda):
    """With 131 071 value heads the 64 token rows of a head span what the
    chunked kernel's 32-bit offsets reach; with more, d = 128 runs in the
    generic kernel. The heads at both ends against a pool of them alone, over
    two calls (the second from the stored state of the first)."""
    d, n = 128, 8
    if kind == "fp32":
        layout, tol = D.damp_layout_init(d, d, 0, D.DAMP_STATE_FP32), 1e-6
    else:  # one code of 255 apart in up to 1e-4 of the values (measured: 5e-5)
        layout, tol = D.damp_layout_init(d, d, 16), 1e-4
    gen = torch.Generator(device="cuda").manual_seed(841)
    slots = torch.zeros(1, dtype=torch.int32, device="cuda")
    ends = torch.cat([torch.arange(n), torch.arange(HV - n, HV)]).cuda()
    pools = [D.Pool(layout, 1, 1, h) for h in (HV, 2 * n)]
    for pool in pools:
        D.damp_pool_reset_slots(pool, 0, slots)
    fn = D.damp_state_prefill_kda if kda else D.damp_state_prefill_gdn
    for _ in range(2):
        x = {m: torch.randn((1, T, HV, d), generator=gen, device="cuda") for m in "qkv"}
        for m in "qk":
            x[m] /= x[m].norm(dim=-1, keepdim=True)
        x["g"] = -torch.rand((1, T, HV, d) if kda else (1, T, HV), generator=gen, device="cuda")
        x["beta"] = torch.rand((1, T, HV), generator=gen, device="cuda")
        o = []
        for pool, pick in zip(pools, (lambda t: t, lambda t: t[:, :, ends])):
            a = {m: pick(t).to(torch.bfloat16).contiguous() for m, t in x.items()}
            o.append(fn(pool, 0, slots, a["q"], a["k"], a["v"], a["g"], a["beta"]))
        assert rel_l2(o[0][:, :, ends].cpu(), o[1].cpu()) <= tol
    S = [D.damp_state_unpack(pool, 0, slots)[0] for pool in pools]
    assert rel_l2(S[0][ends].cpu(), S[1].cpu()) <= tol


PREFILL_FORMATS = {"fp32": (orc.KIND_FP32, 0, None), "default": (orc.KIND_MIXED, 16, None),
                   "default_k0": (orc.KIND_MIXED, 0, None),
                   "int8_h32": (orc.KIND_MIXED, 16, orc.FMT_PAPER),
                   "int8_g32": (orc.KIND_MIXED, 16, orc.FMT_PAPER_PLAIN),
                   "int4": (orc.KIND_MIXED, 16, orc.FMT_INT4),
                   "int4_h32": (orc.KIND_MIXED, 16, orc.FMT_INT4_H32),
                   "fp8": (orc.KIND_MIXED, 16, orc.FMT_FP8),
                   "nvfp4": (orc.KIND_MIXED, 16, orc.FMT_NVFP4)}


@pytest.mark.parametrize("B", [5, 131])
@pytest.mark.parametrize("kda", [False, True])
@pytest.mark.parametrize("name", list(PREFILL_FORMATS))
def test_prefill_formats_at_both_launch_shapes(name, kda, B):
    """d = 128 in every storage format, with up to 256 tiles (staging waves of
    their own) and with more (four waves, the tile's transit in the memory of
    the staged chunks): a partial last chunk, permuted channels, scattered
    slots, a padded and an out-of-range request, and slots that no request
    names, which keep their bytes."""
    kind, k_hi, fmt = PREFILL_FORMATS[name]
    d, HV, T, n_slots = 128, 2, 37, B + 3
    HK = HV if kda else 1
    seed = 851 + B
    _say(f"prefill {name} kda={kda} B={B}")
    slots = inputs.slot_order(seed, n_slots, B)
    slots[1], slots[3] = -1, n_slots
    live = (slots >= 0) & (slots < n_slots)
    perm = inputs.random_perms(seed, HV, d)
    ref = orc.Pool(kind, d, d, k_hi, 1, n_slots, HV, fmt=fmt)
    # the states of every slot, those of no request among them
    orc.pack(ref, 0, np.arange(n_slots), inputs.synthetic_states(seed, n_slots, HV, d), perm)
    before = ref.buf.copy()
    gpool = gpu_pool_from(ref, D)
    inp = inputs.as_prefill(inputs.decode_inputs(seed, T, B, HK, HV, d, kda=kda))
    o_gpu, o_ref = _run(kda, ref, gpool, slots, inp, perm, scale=0.5)
    host = gpool.buffer.cpu().numpy()
    err = rel_l2(o_gpu, o_ref)
    stats = compare_tiles(host, ref, f"prefill {name}", s16_exact_min=0.99)
    _say(f"  o rel-L2 {err:.2e}  {stats}")
    # identical starting bytes and fp32 from there: only the order of the sums
    assert err <= 1e-6
    assert (o_gpu[~live] == 0).all()
    idle = np.setdiff1d(np.arange(n_slots), slots[live])
    st = ref.slot_stride
    for s in idle:
        assert np.array_equal(host[s * st:(s + 1) * st], before[s * st:(s + 1) * st])


@pytest.mark.parametrize("B", [2, 129])
@pytest.mark.parametrize("power", [28, -20, -60, -90])
@pytest.mark.parametrize("kda", [False, True])
def test_prefill_scale_of_queries(kda, power, B):
    """o is linear in q: its scale costs no precision, KDA's decays as in the
    test of the state's scale."""
    HV, T, seed = 2, 40, 861
    ref, gpool, inp = _fp32_case(kda, B, HV, T, seed, inputs.synthetic_states(seed, B, HV, 128))
    inp["q"] = _scale_bf16(inp["q"], 2.0 ** power)
    if kda:
        g = inp["g"].copy()
        g[..., 3::16] = _bits(-79 * np.log(2.0) / 8)
        inp["g"] = g
    o_gpu, o_ref = _run(kda, ref, gpool, np.arange(B), inp, None)
    err = rel_l2(o_gpu, o_ref)
    _say(f"  kda={kda} 2^{power} B={B}: o rel-L2 {err:.2e}")
    assert err <= 1e-6


@pytest.mark.parametrize("B", [2, 257])
@pytest.mark.parametrize("norm,T", [(1.0, 40), (64.0, 6)])
def test_prefill_kda_wide_operands_beside_steep_channels(norm, T, B):
    """beta in (0, 2) and factors above one, where a chunk's |A| is looked at:
    within its bound (keys of norm 1) the chunk stays in matrix form, beyond it
    (norm 64) it runs token by token, with steep channels staged in it either
    way. Six tokens of the larger keys grow the state to about 1e19, and its
    rounding with it."""
    HV, seed = 1, 871
    ref, gpool, inp = _fp32_case(True, B, HV, T, seed, inputs.synthetic_states(seed, B, HV, 128))
    inp["k"] = _scale_bf16(inp["k"], norm)
    inp["beta"] = _scale_bf16(inp["beta"], 2.0)
    g = inp["g"].copy()
    g[..., 11] = _bits(0.125)
    g[..., 40:43] = _bits(-20.0)
    inp["g"] = g
    o_gpu, o_ref = _run(True, ref, gpool, np.arange(B), inp, None)
    state = gpool.buffer.cpu().numpy().view(np.float32)
    err, s_err = rel_l2(o_gpu, o_ref), rel_l2(state, ref.buf.view(np.float32))
    _say(f"  norm {norm} B={B}: o rel-L2 {err:.2e} state rel-L2 {s_err:.2e}")
    tol = 1e-6 if norm == 1.0 else 1e-4
    assert np.isfinite(o_ref).all() and err <= tol and s_err <= tol
