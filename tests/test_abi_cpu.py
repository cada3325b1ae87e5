"""The C ABI on the host, without a GPU: the library loads, exports every
function include/sps.h declares, and rejects invalid arguments with status
codes before any HIP call."""
import ctypes
import os
import re

import pytest

from paper_2302_01318_amd import configs

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2302_01318_amd", "libsps.so")


@pytest.fixture(scope="module")
def sps():
    if not os.path.exists(LIB):
        from paper_2302_01318_amd import build
        build.build()
    from paper_2302_01318_amd import sps as mod
    return mod


def declared_functions():
    text = open(os.path.join(ROOT, "include", "sps.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(sps_[a-z0-9_]+)\s*\(", text)))


def test_every_declared_function_is_exported(sps):
    names = declared_functions()
    assert len(names) >= 19
    for n in names:
        assert hasattr(sps.lib, n), n
    assert sorted(sps.EXPORTS) == names


def test_status_strings(sps):
    assert sps.lib.sps_status_string(0) == b"ok"
    assert sps.lib.sps_status_string(5) == b"HIP runtime error"
    assert sps.lib.sps_abi_version() == 3


def test_config_validation_and_sizes(sps):
    from paper_2302_01318_amd import configs
    good = sps.config_of(configs.SEVENTY_B)
    assert sps.lib.sps_weight_bytes(ctypes.byref(good)) >= configs.SEVENTY_B.n_params() * 2
    for field, bad in [("d_model", 100), ("head_dim", 96), ("vocab", 1), ("vocab", 1 << 24), ("d_ff", 48),
                       ("ffn_kind", 2), ("dtype", 3), ("n_layers", 0)]:
        c = sps.config_of(configs.SEVENTY_B)
        setattr(c, field, bad)
        assert sps.lib.sps_weight_bytes(ctypes.byref(c)) == 0, field
        h = ctypes.c_void_p()
        assert sps.lib.sps_model_create(ctypes.byref(c), ctypes.c_void_p(1), ctypes.byref(h)) == 2
    assert sps.lib.sps_kv_bytes(ctypes.byref(good), 1, 100) == 0          # T_cap % 32
    assert sps.lib.sps_kv_bytes(ctypes.byref(good), 1, 2304) == 80 * 2 * 64 * 2304 * 128 * 2
    assert sps.lib.sps_workspace_bytes(ctypes.byref(good), 0, 5, 2304) == 0
    # KV capacity at most 2^22 positions
    assert sps.lib.sps_kv_bytes(ctypes.byref(good), 1, 1 << 22) == 80 * 2 * 64 * (1 << 22) * 128 * 2
    assert sps.lib.sps_kv_bytes(ctypes.byref(good), 1, (1 << 22) + 32) == 0
    assert sps.lib.sps_workspace_bytes(ctypes.byref(good), 1, 5, (1 << 22) + 32) == 0
    assert sps.lib.sps_workspace_bytes(ctypes.byref(good), 1, 5, 1 << 22) > 0
    h = ctypes.c_void_p()
    assert sps.lib.sps_kv_create(ctypes.byref(good), 1, (1 << 22) + 32, ctypes.c_void_p(1), ctypes.c_void_p(1),
                                 ctypes.byref(h)) == 2 and not h.value


def test_fp8_config_and_slots(sps):
    from paper_2302_01318_amd import configs
    s70 = configs.SEVENTY_B
    b16 = sps.config_of(s70)
    f8 = sps.config_of(s70.with_(dtype="fp8"))
    nb, n8 = sps.lib.sps_weight_bytes(ctypes.byref(b16)), sps.lib.sps_weight_bytes(ctypes.byref(f8))
    # projections halve; the bf16 embedding (V x d) and the scales stay
    V, d = s70.vocab, s70.d_model
    assert n8 < nb and abs((nb - V * d * 2) / 2 - (n8 - V * d * 2)) < 0.001 * nb
    # FP8 needs 64-deep contractions: d_model, heads x head_dim and d_ff multiples of 64
    for field, bad in [("d_model", 96), ("d_ff", 96)]:
        c = sps.config_of(s70.with_(dtype="fp8"))
        setattr(c, field, bad)
        assert sps.lib.sps_weight_bytes(ctypes.byref(c)) == 0, field
    c = sps.config_of(configs.ModelShape("x", 96, 1, 1, 64, 128, 100, "gelu", "bf16"))
    assert sps.lib.sps_weight_bytes(ctypes.byref(c)) > 0
    c.dtype = 2
    assert sps.lib.sps_weight_bytes(ctypes.byref(c)) == 0
    # slots: FP8 projections carry row scales right after their codes; bf16 ones none
    o, n, sc = sps.weight_slot(s70.with_(dtype="fp8"), "w1", 3)
    assert n == 32768 * 8192 and sc >= o + n and sc - (o + n) < 256
    o2, n2, sc2 = sps.weight_slot(s70, "w1", 3)
    assert n2 == 2 * n and sc2 == 0
    assert sps.weight_slot(s70.with_(dtype="fp8"), "wq", 0)[0] == sps.weight_slot(s70.with_(dtype="fp8"), "wv", 0)[0]
    for layer in (-1, 80):
        with pytest.raises(sps.SPSError):
            sps.weight_slot(s70, "wo", layer)
    with pytest.raises(sps.SPSError):
        sps.weight_slot(s70, "w3", 0)                  # GELU model: no W3
    P = ctypes.c_void_p
    assert sps.lib.sps_fp8_decode(P(16), 17, P(16), None) == 1
    assert sps.lib.sps_fp8_decode(P(8), 16, P(16), None) == 1
    assert sps.lib.sps_fp8_decode(None, 16, P(16), None) == 1


def test_invalid_arguments_return_codes(sps):
    Ph = sps.Philox(0, 0)
    P = ctypes.c_void_p
    one = P(1)
    # accept_resample: bad K, bad V, null outputs
    assert sps.lib.sps_accept_resample(one, one, one, None, Ph, 1, -1, 10, one, one, None) == 1
    assert sps.lib.sps_accept_resample(one, one, one, None, Ph, 1, 64, 10, one, one, None) == 1
    assert sps.lib.sps_accept_resample(one, one, one, None, Ph, 1, 2, 1, one, one, None) == 1
    assert sps.lib.sps_accept_resample(one, one, one, None, Ph, 1, 2, 10, None, one, None) == 1
    assert sps.lib.sps_accept_resample(None, one, one, None, Ph, 1, 2, 10, one, one, None) == 1
    # forward / verify / draft / commit with null handles
    assert sps.lib.sps_forward(None, None, one, 5, 1, 5, 0, None, one, 1 << 30, None) == 1
    S = sps.sampling_of
    assert sps.lib.sps_verify_step(None, None, one, 1, 4, S(1.0), None, None, None, one, 1 << 30, None) == 1
    assert sps.lib.sps_verify_step(None, None, one, 1, -1, S(1.0), None, None, None, one, 1 << 30, None) == 1
    assert sps.lib.sps_draft_step(None, None, one, 1, 4, S(-1.0), Ph, one, one, one, 1 << 30, None) == 1
    assert sps.lib.sps_commit(None, one, one, one, 1, 4, one, None, None, 0, None) == 1
    assert sps.lib.sps_pack_weight(None, 0, 0, one, one, None) == 2
    assert sps.lib.sps_philox_uniforms(Ph, 0, 1, 1, None, None) == 1
    assert sps.lib.sps_softmax(one, 1, 1, S(1.0), one, None) == 1
    # sampling parameters: negative top_k, top_p outside [0, 1] or NaN; modifiers beyond the supported vocabulary
    assert sps.lib.sps_softmax(one, 1, 1000, S(1.0, -1, 1.0), one, None) == 1
    assert sps.lib.sps_softmax(one, 1, 1000, S(1.0, 0, 1.5), one, None) == 1
    assert sps.lib.sps_softmax(one, 1, 1000, S(1.0, 0, float("nan")), one, None) == 1
    assert sps.lib.sps_softmax(one, 1, 1000, S(float("inf")), one, None) == 1
    assert sps.lib.sps_softmax(one, 1, 40000, S(1.0, 5, 1.0), one, None) == 4
    assert sps.lib.sps_softmax(one, 1, 40000, S(1.0, 0, 0.9), one, None) == 4
    assert sps.lib.sps_device_error(None, 0, None) == 1
    # streaming-read helper: zero, ragged or misaligned sizes, null pointers
    sixteen = P(16)
    assert sps.lib.sps_stream_read(sixteen, 0, sixteen, None) == 1
    assert sps.lib.sps_stream_read(sixteen, 24, sixteen, None) == 1
    assert sps.lib.sps_stream_read(P(8), 32, sixteen, None) == 1
    assert sps.lib.sps_stream_read(None, 32, sixteen, None) == 1
    assert sps.lib.sps_stream_read(sixteen, 32, None, None) == 1


def test_handles_and_shape_checks(sps):
    from paper_2302_01318_amd import configs
    tiny = sps.config_of(configs.TINY_TARGET)
    other = sps.config_of(configs.TINY_DRAFT)
    m, kv, kv2 = ctypes.c_void_p(), ctypes.c_void_p(), ctypes.c_void_p()
    one = ctypes.c_void_p(1)
    assert sps.lib.sps_model_create(ctypes.byref(tiny), one, ctypes.byref(m)) == 0
    assert sps.lib.sps_kv_create(ctypes.byref(tiny), 2, 64, one, one, ctypes.byref(kv)) == 0
    assert sps.lib.sps_kv_create(ctypes.byref(other), 2, 64, one, one, ctypes.byref(kv2)) == 0
    bad = ctypes.c_void_p()
    assert sps.lib.sps_kv_create(ctypes.byref(tiny), 2, 65, one, one, ctypes.byref(bad)) == 2
    assert bad.value is None
    need = sps.lib.sps_workspace_bytes(ctypes.byref(tiny), 2, 5, 64)
    # workspace too small, batch mismatch, too many tokens per sequence, cache of another model
    assert sps.lib.sps_forward(m, kv, one, 5, 2, 5, 0, None, one, need - 1, None) == 3
    assert sps.lib.sps_forward(m, kv, one, 5, 3, 5, 0, None, one, need, None) == 2
    assert sps.lib.sps_forward(m, kv, one, 65, 2, 65, 0, None, one, 1 << 40, None) == 2
    assert sps.lib.sps_forward(m, kv2, one, 5, 2, 5, 0, None, one, 1 << 40, None) == 2
    assert sps.lib.sps_kv_write(kv, 0, 0, 60, 8, one, one, None) == 3
    assert sps.lib.sps_kv_write(kv, 4, 0, 0, 8, one, one, None) == 1
    sps.lib.sps_model_destroy(m)
    sps.lib.sps_kv_destroy(kv)
    sps.lib.sps_kv_destroy(kv2)


def test_workspace_requests_no_call_admits(sps):
    """sps_workspace_bytes refuses at once what no call can use (more than 64
    tokens per sequence, more than 160 rows), and covers every smaller
    request it admits (the draft step's 2-then-1 token layout included)."""
    import ctypes
    import time
    c = ctypes.byref(sps.config_of(configs.SEVENTY_B))
    t0 = time.time()
    assert sps.lib.sps_workspace_bytes(c, 1, 2 ** 31 - 1, 2112) == 0
    assert sps.lib.sps_workspace_bytes(c, 2 ** 31 - 1, 1, 2112) == 0
    assert time.time() - t0 < 1.0
    assert sps.lib.sps_workspace_bytes(c, 1, 65, 2112) == 0
    assert sps.lib.sps_workspace_bytes(c, 3, 54, 2112) == 0
    assert sps.lib.sps_workspace_bytes(c, 1, 64, 2112) > 0
    d = ctypes.byref(sps.config_of(configs.DRAFT_70B))
    for B in range(1, 81):
        two = sps.lib.sps_workspace_bytes(d, B, 2, 2112)
        assert two >= sps.lib.sps_workspace_bytes(d, B, 1, 2112) > 0


def test_generator_refuses_a_draft_of_another_vocabulary(sps):
    """The draft's p rows are read at the target's vocabulary stride: a draft
    with another vocabulary is refused before anything is allocated."""
    class Fake:
        def __init__(self, shape):
            self.shape = shape
    with pytest.raises(ValueError, match="vocabulary"):
        sps.Generator(Fake(configs.TINY_TARGET), Fake(configs.TINY_DRAFT.with_(vocab=1000)), 1, 64, 4,
                      device="cpu")


@pytest.mark.parametrize("B,T_cap,at_most,want", [
    (1, 256, None, 160), (2, 256, None, 80), (3, 256, None, 53), (1, 32, None, 64), (1, 96, None, 96),
    (1, 256, 64, 64), (1, 256, 100, 100), (1, 256, 7, 7), (1, 256, 0, 1), (1, 256, 1000, 160), (2, 256, 64, 64),
    (4, 256, 64, 40), (1, 1 << 20, None, 64), (1, 1 << 20, 32, 32)])
def test_generator_prefill_chunk(sps, monkeypatch, B, T_cap, at_most, want):
    """prefill_chunk bounds the tokens of a prefill chunk, and the Generator's
    workspace with them; by default a chunk has as many as 160 rows hold, but
    past 64 no more than the cache and no more scratch than PREFILL_BYTES."""
    shape = configs.DRAFT_70B if T_cap > 256 else configs.TINY_TARGET
    assert sps.prefill_tokens([shape], B, T_cap, at_most) == want
    if T_cap > 256:
        return

    class Fake:
        pass
    model = Fake()
    model.shape = shape
    monkeypatch.setattr(sps, "KVCache", lambda *a: None)          # wants device memory
    args = {} if at_most is None else {"prefill_chunk": at_most}
    gen = sps.Generator(model, None, B, T_cap, 4, device="cpu", **args)
    c = ctypes.byref(sps.config_of(shape))
    assert gen.chunk == want
    assert gen.ws_t.numel() == max(sps.lib.sps_workspace_bytes(c, B, max(min(want, 64), 5), T_cap),
                                   sps.lib.sps_prefill_workspace_bytes(c, B, want, T_cap))
