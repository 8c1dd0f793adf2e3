"""Host-side checks of the C-ABI library: it loads, exports every declared symbol,
and its host-only entry points agree with the oracle.  No GPU work is launched."""
import array
import ctypes
import math
import os
import re

import numpy as np
import pytest

from oracle import cache as ocache
from oracle import sampler
from paper_2501_04012_amd import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_symbols():
    text = open(os.path.join(ROOT, "include", "flexdenoise.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(fc_[a-z0-9_]+)\s*\(", text)))


def test_library_exports_every_declared_symbol(fc):
    lib = ctypes.CDLL(fc.binding.LIB_PATH)
    names = declared_symbols()
    assert "fc_denoise_step" in names and "fc_denoise_resume" in names and len(names) >= 15
    for n in names:
        assert hasattr(lib, n), n
    # and the binding wraps each of them under the same name
    for n in names:
        assert hasattr(fc.binding, n) or n in ("fc_status_string", "fc_last_error"), n
    # the profile categories are the ones the header lists, in its order
    text = open(os.path.join(ROOT, "include", "flexdenoise.h")).read()
    macro = text[text.index("#define FC_PROFILE_CATEGORY_NAMES"):].split("int fc_profile_enable")[0]
    listed = " ".join(re.findall(r'"([^"]*)"', macro)).split()
    assert fc.fc_profile_categories() == len(listed)
    assert [fc.fc_profile_category_name(i) for i in range(len(listed))] == listed


def test_schedule_coefficients_match_oracle(fc):
    sched = synth.Schedule()
    for step in (1, 10, 25, 49, 50):
        coef, t = fc.fc_schedule_coefficients(sched, step)
        ot, a_t, a_p = sampler.step_coefficients(sched, step)
        assert t == ot
        want = [math.sqrt(a_t), math.sqrt(1 - a_t), math.sqrt(a_p), math.sqrt(1 - a_p)]
        np.testing.assert_allclose(coef, want, rtol=2e-6, atol=1e-7)
    coef, t = fc.fc_schedule_coefficients(sched, 50)
    assert t == 0 and coef[2] == 1.0 and coef[3] == 0.0


def test_flow_euler_coefficients_match_oracle(fc):
    from dataclasses import replace
    sched = replace(synth.Schedule(), sampler=synth.SAMPLER_FLOW_EULER)
    for step in (1, 2, 25, 50):
        coef, t = fc.fc_schedule_coefficients(sched, step)
        ot, sig, nxt = sampler.flow_step_sigmas(sched, step)
        assert t == ot
        np.testing.assert_allclose(coef, [1.0, 0.0, 1.0, nxt - sig], rtol=1e-6, atol=0)
    with pytest.raises(fc.FlexDenoiseError) as e:
        fc.fc_schedule_coefficients(replace(sched, num_steps=30), 1)      # 1000 % 30 != 0
    assert e.value.status == -6
    with pytest.raises(fc.FlexDenoiseError) as e:
        fc.fc_schedule_coefficients(replace(sched, sampler=7), 1)
    assert e.value.status == -3


def test_schedule_errors_are_status_codes(fc):
    from dataclasses import replace
    sched = synth.Schedule()
    for bad in (0, 51, -3):
        with pytest.raises(fc.FlexDenoiseError) as e:
            fc.fc_schedule_coefficients(sched, bad)
        assert e.value.status == -3
    for bad_eta in (-0.1, 1.5):
        with pytest.raises(fc.FlexDenoiseError) as e:
            fc.fc_schedule_coefficients(replace(sched, eta=bad_eta), 1)
        assert e.value.status == -3
    with pytest.raises(fc.FlexDenoiseError) as e:
        fc.fc_schedule_coefficients(replace(sched, eta=0.5, sampler=synth.SAMPLER_FLOW_EULER), 1)
    assert e.value.status == -6
    # eta > 0 keeps sqrt(1 - abar_prev - sigma^2) on the eps direction
    coef, _ = fc.fc_schedule_coefficients(replace(sched, eta=0.5), 20)
    _, a_t, a_p = sampler.step_coefficients(sched, 20)
    sg = sampler.ddim_sigma(a_t, a_p, 0.5)
    np.testing.assert_allclose(coef[3], math.sqrt(1 - a_p - sg * sg), rtol=2e-6)


def test_model_configuration_errors_and_weight_counts(fc):
    from dataclasses import replace
    tiny = synth.WORKLOADS["cfg1"].model
    # separate text modulation exists only where the text rows are part of the sequence
    with pytest.raises(fc.FlexDenoiseError) as e:
        fc.fc_model_create(replace(tiny, attn_mode=synth.ATTN_FACTORIZED_CROSS, text_adaln=1))
    assert e.value.status == -2
    with pytest.raises(fc.FlexDenoiseError) as e:
        fc.fc_model_create(replace(tiny, attn_mode=synth.ATTN_FULL3D_CONCAT, text_adaln=2))
    assert e.value.status == -2
    D = tiny.hidden
    full = replace(tiny, attn_mode=synth.ATTN_FULL3D_CONCAT)
    assert synth.weight_count(replace(full, text_adaln=1)) - synth.weight_count(full) == tiny.depth * 6 * D * (D + 1)


def test_weight_spec_matches_library_count_formula():
    # closed-form parameter counts: cfg-2 block has 29 D^2 + biases; cfg-4 block 18 D^2 + biases
    c2 = synth.WORKLOADS["cfg2"].model
    D, M = c2.hidden, c2.mlp_dim
    blk = 9 * D * D + 9 * D + 2 * (3 * D * D + 3 * D + D * D + D) + (D * D + D) + (2 * D * D + 2 * D) + (D * D + D) \
        + 2 * D * M + M + D
    head = 256 * D + D + D * D + D + 4096 * D + D + 16 * D + D + 2 * D * D + 2 * D + D * 16 + 16
    assert synth.weight_count(c2) == blk + head


def test_flop_accounting_matches_hand_counts():
    f2 = synth.forward_flops(synth.WORKLOADS["cfg2"].model)
    assert abs(f2["block_gemm"] + f2["block_attention"] - 203.8e9) / 203.8e9 < 5e-3
    f4 = synth.forward_flops(synth.WORKLOADS["cfg4"].model)
    assert abs(f4["block_attention"] - 3.883e12) / 3.883e12 < 1e-3
    assert abs(f4["block_gemm"] + f4["block_attention"] - 7.91e12) / 7.91e12 < 2e-3


def test_key_frame_selection_matches_oracle(fc):
    """fc_cache_select_key_frames is host logic: same maps as the oracle on random and on
    constructed similarity matrices, thresholds 0.9 and 0.99."""
    rng = np.random.default_rng(3)
    base = rng.standard_normal((5, 6, 6, 4))
    for T in (1, 2, 7, 24, 64):
        frames = np.stack([base[rng.integers(5)] + 0.06 * rng.standard_normal((6, 6, 4)) for _ in range(T)])
        sim = ocache.frame_similarity(frames).astype(np.float32)
        for thr in (0.9, 0.99):
            want = ocache.select_key_frames(sim, np.float32(thr))
            got = fc.fc_cache_select_key_frames(sim, thr)
            assert np.array_equal(got, want), (T, thr)
    chain = np.array([[1.0, 0.995, 0.98], [0.995, 1.0, 0.995], [0.98, 0.995, 1.0]], dtype=np.float32)
    assert np.array_equal(fc.fc_cache_select_key_frames(chain, 0.99), [0, 2, 2])
    assert fc.fc_cache_workspace_bytes(0) >= 4096 and fc.fc_cache_workspace_bytes(64) >= 64 * 64 * 8


@pytest.mark.parametrize("src", [
    [0, 3, -1, 2], (0, 3, -1, 2), [0.0, 3.9, -1.0, 2.0], [np.int64(0), np.float32(3.0), -1, True],
    np.array([0, 3, -1, 2]), np.array([0, 3, -1, 2], dtype=np.int8), np.array([0.0, 3.0, -1.0, 2.0]), b"\x00\x03\x01\x02",
    bytearray(b"\x00\x03\x01\x02"), bytes(64), range(4), [2 ** 32 + 1, -2 ** 31, 2 ** 31, 0], ["0", "3", "-1", "2"], [0, 3], [],
    array.array("b", [0, 3, -1, 2]), array.array("d", [0.0, 3.0, -1.0, 2.0]), np.array([2 ** 32 - 1, 1], dtype=np.uint32)])
@pytest.mark.parametrize("once", [False, True])
def test_decompress_source_codes(monkeypatch, src, once):
    """Every iterable of numbers gives int(v) per frame, the rest zero, also one that can be walked only once."""
    from paper_2501_04012_amd import binding
    frames, seen = max(len(src), 4), {}

    class Library:
        def fc_cache_decompress(self, first, base, n_base, alpha, extra, n_extra, codes, frames, *rest):
            address = codes if isinstance(codes, int) else ctypes.addressof(codes)
            seen["codes"] = list((ctypes.c_int32 * frames).from_address(address))
            return 0

    monkeypatch.setattr(binding, "_lib", Library())
    want = list((ctypes.c_int32 * frames)(*[int(v) for v in src]))
    binding.fc_cache_decompress(None, None, 0, 1.0, None, 0, iter(src) if once else src, frames, 1, None, stream=1)
    assert seen["codes"] == want
    with pytest.raises(IndexError):
        binding.fc_cache_decompress(None, None, 0, 1.0, None, 0, [0] * 5, 4, 1, None, stream=1)


@pytest.mark.parametrize("private", [True, False])
def test_current_stream_handle(monkeypatch, private):
    """With torch's own names for the device and the stream's handle, and without them."""
    import torch
    from paper_2501_04012_amd import binding
    monkeypatch.setattr(torch.cuda, "init", lambda: None)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: type("S", (), {"cuda_stream": 3})())
    if private:
        monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 1, raising=False)
        monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 10 + device, raising=False)
    else:
        monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    monkeypatch.setattr(binding, "_current_stream", None)
    assert binding._stream(None) == (11 if private else 3)
    assert binding._stream(7) == 7 and binding._stream(0) is None


def test_forked_child_asks_for_the_device_again(monkeypatch):
    """torch raises in a child forked after the device was used; a handle kept from the parent would bypass that."""
    from paper_2501_04012_amd import binding
    monkeypatch.setattr(binding, "_current_stream", lambda: 5)
    pid = os.fork()
    if pid == 0:
        os._exit(0 if binding._current_stream is None else 1)
    assert os.waitstatus_to_exitcode(os.waitpid(pid, 0)[1]) == 0
    assert binding._stream(None) == 5


@pytest.mark.parametrize("call,args,status", [
    ("fc_cache_decompress", (None, None, 0, 1.0, None, 0, [0], 1, 4, None), -1),
    ("fc_cache_decompress", ("t", None, 0, 1.0, None, 0, [1], 1, 4, "t"), -3),                 # a frame the entry does not hold
    ("fc_cache_decompress", ("t", None, 0, 1.0, None, 0, [0] * 257, 257, 4, "t"), -6),
    ("fc_cache_decompress", ("t", None, 0, 1.0, None, 0, [0], 1, 0, "t"), 0),                   # nothing to do: no launch
    ("fc_cache_stitch", ("t", "t", None, None, "t", 4, 4), -1),
    ("fc_cache_stitch", ("t", "t", "t", None, "t", 4, 0), -3),
    ("fc_cache_stitch", ("t", "t", "t", "t", "t", 0, 4), 0),
    ("fc_cache_alpha", ("t", "t", "t", 0, 4, "t", "t"), -3),
    ("fc_cache_alpha", ("t", "t", "t", 1, 4, "t", "t"), -4),
    ("fc_cache_frame_similarity", (None, 1, 4, "t", "t"), -1),
    ("fc_cache_frame_similarity", ("t", 1, 4, "t", "t"), -4)])
@pytest.mark.parametrize("native", [True, False])
def test_cache_calls_by_both_routes(monkeypatch, call, args, status, native):
    """The CPython route and the ctypes one give the same status for the same arguments."""
    import torch
    from paper_2501_04012_amd import binding
    t = torch.zeros(16)
    args = [t if isinstance(a, str) else a for a in args]
    if not native:
        monkeypatch.setattr(binding, "_fast_lib", None)
    if status == 0:
        getattr(binding, call)(*args, stream=1)
        return
    with pytest.raises(binding.FlexDenoiseError) as e:
        getattr(binding, call)(*args, stream=1)
    assert e.value.status == status and call in str(e.value)


def test_native_route_leaves_other_arguments_to_ctypes():
    import torch
    from paper_2501_04012_amd import binding
    t = torch.zeros(16)
    plain = [t, None, 0, 1.0, None, 0, [0], 1, 0, t, None]
    assert binding._fast.fc_cache_decompress(*plain) == 0
    for at, other in ((0, np.zeros(4, np.float32)), (2, np.int64(0)), (2, False), (2, 2 ** 31), (3, 1), (3, np.float32(1)), (6, [0, 0]),
                      (6, np.zeros(1, np.int64)), (6, [np.int64(0)]), (6, [2 ** 31]), (6, iter([0])), (7, 0), (8, 2 ** 63), (8, 0.0),
                      (10, "x")):
        with pytest.raises(TypeError):
            binding._fast.fc_cache_decompress(*(plain[:at] + [other] + plain[at + 1:]))
    with pytest.raises(TypeError):
        binding._fast.fc_cache_decompress(*plain[:-1])


def test_package_imports_without_the_native_route():
    """Every cache call has its ctypes form: the package works where the extension was not built for this interpreter."""
    import subprocess
    import sys
    code = """
import sys
sys.modules["paper_2501_04012_amd._pycall"] = None        # an import of it fails
import torch
import paper_2501_04012_amd as fc
assert fc.binding._fast is None and fc.binding._fast_lib is None
t = torch.zeros(16)
fc.fc_cache_decompress(t, None, 0, 1.0, None, 0, [0], 1, 0, t, stream=1)
fc.fc_cache_stitch(t, t, t, t, t, 0, 4, stream=1)
for call, args, status in ((fc.fc_cache_alpha, (t, t, t, 1, 4, t, t), -4), (fc.fc_cache_frame_similarity, (t, 1, 4, t, t), -4)):
    try:
        call(*args, stream=1)
    except fc.FlexDenoiseError as e:
        assert e.status == status
    else:
        raise AssertionError(call)
"""
    subprocess.run([sys.executable, "-c", code], cwd=ROOT, check=True)


def test_native_route_is_built_for_one_interpreter():
    import sysconfig
    from paper_2501_04012_amd import binding, build
    assert build.PYCALL_PATH.endswith(sysconfig.get_config_var("EXT_SUFFIX")) and "cpython" in os.path.basename(build.PYCALL_PATH)
    assert binding._fast.__file__ == build.PYCALL_PATH


def test_build_without_a_host_compiler(monkeypatch, tmp_path, capsys):
    """The library is built all the same, an extension of an earlier build does not stay."""
    from paper_2501_04012_amd import build
    calls = []

    def run(cmd):
        if cmd[0] == "no-such-compiler":
            raise FileNotFoundError(cmd[0])
        calls.append(cmd)
        return ""
    monkeypatch.setenv("CXX", "no-such-compiler")
    monkeypatch.setattr(build, "_run", run)
    for name in ("OBJ_DIR", "LIB_PATH", "PYCALL_PATH"):
        monkeypatch.setattr(build, name, str(tmp_path / os.path.basename(getattr(build, name))))
    (tmp_path / os.path.basename(build.PYCALL_PATH)).write_bytes(b"old")
    assert build.build(force=True) == build.LIB_PATH and len(calls) == len(build.SOURCES) + 1
    assert not os.path.exists(build.PYCALL_PATH) and "ctypes" in capsys.readouterr().err
