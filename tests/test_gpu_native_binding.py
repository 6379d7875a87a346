"""The binding's CPython module: the same results as the ctypes path (which a call with its stream named takes), and the
calls it does not take, which go there."""
import ctypes
import math
import os
import shutil
import subprocess
import sys
import sysconfig

import pytest
import torch

import paper_2603_17051_amd as A
from paper_2603_17051_amd import binding, build

GOOD = dict(batch=2, heads=2, head_dim=64, grid_h=4, grid_w=8, capacity_frames=4, sink_frames=1, max_chunk_frames=2,
            rope_pairs=(12, 10, 10))


def test_calls_it_does_not_take_are_left_alone():
    cache = A.astro_kvcache_create(host_only=True, **GOOD)
    x, dims = torch.zeros(2, 32, 2, 64, dtype=torch.bfloat16), cache._native_dims
    append = binding._native.append
    assert append(cache.handle, dims, x, x, 1) is None  # not on a device
    assert append(cache.handle, dims, None, x, 1) is None and append(cache.handle, dims, x) is None
    for handle in (None, 7, ctypes.c_void_p(None)):
        assert append(handle, dims, x, x, 1) is None
    for frames in (True, 1.0, -1, 1 << 40, None):
        assert append(cache.handle, dims, x, x, frames) is None
    assert append(cache.handle, dims[:4], x, x, 1) is None
    one = torch.ones(1)
    assert binding._native.loss(one, one, one, one, one, one, 1.0, 1.0, 0.1, None, None, None) is None
    with pytest.raises(TypeError):
        binding._native.bind((1, 2))
    cache.close()


class Answers:
    """The module's functions, and what each of their calls answered."""

    def __init__(self):
        self.module, self.got = binding._native, []

    def __getattr__(self, name):
        def call(*args):
            self.got.append((name, len(args), getattr(self.module, name)(*args)))
            return self.got[-1][2]
        return call


@pytest.fixture
def answers(monkeypatch):
    monkeypatch.setattr(binding, "_native", Answers())
    return binding._native.got


@pytest.mark.gpu
@pytest.mark.parametrize("group", [1, 3])
def test_attention_calls_give_what_the_ctypes_path_gives(group, answers):
    gen = torch.Generator("cuda:0").manual_seed(3)
    draw = lambda b, n: torch.randn((b, n * 32, 2, 64), generator=gen, device="cuda:0").bfloat16()
    k0, v0 = draw(2, 2), draw(2, 2)
    q, k, v, do = (draw(2 * group, 2) for _ in range(4))
    results = []
    for stream in (None, torch.cuda.current_stream()):
        cache = A.astro_kvcache_create(**GOOD)
        A.astro_kvcache_append(cache, k0, v0, 2, stream=stream)
        need = max(A.astro_group_attn_workspace_bytes(cache, 2, group))
        ws = torch.empty(max(need, A.astro_chunk_attn_bwd_full_workspace_bytes(cache, 2)), dtype=torch.uint8, device="cuda:0")
        out, lse = torch.empty_like(q), torch.empty((2 * group, 2, 64), device="cuda:0")
        g = [torch.empty(q.shape, device="cuda:0") for _ in range(3)]
        ring = [torch.zeros((2, 4 * 32, 2, 64), device="cuda:0") for _ in range(2)]
        if group == 1:
            got = A.astro_chunk_attn_fwd(cache, q, k, v, 2, out, lse, ws, stream=stream)
            got += A.astro_chunk_attn_bwd(cache, q, k, v, out, lse, do, 2, *g, ws, stream=stream)
            got = [x.clone() for x in got]
            got += A.astro_chunk_attn_bwd_full(cache, q, k, v, out, lse, do, 2, *g, *ring, ws, stream=stream)
        else:
            got = A.astro_group_attn_fwd(cache, q, k, v, 2, group, out, lse, ws, stream=stream)
            got += A.astro_group_attn_bwd(cache, q, k, v, out, lse, do, 2, group, *g, ws, stream=stream)
        # the module took every one of these calls, or (stream named) was not asked
        took = [("append", 5, 0), ("fwd", 10, 0), ("bwd", 14, 0)] + ([("bwd", 17, 0)] if group == 1 else [])
        assert answers == (took if stream is None else [])
        results.append([x.clone() for x in got] + [cache.k_storage.clone()])
        # refused on both ways
        for change in (dict(q=q.float()), dict(q=q[:1]), dict(q=q.transpose(0, 1)), dict(q=q.cpu()), dict(lse=lse[:1] if group > 1 else None, out=out[:1])):
            a = dict(q=q, out=out, lse=lse)
            a.update(change)
            with pytest.raises(ValueError):
                A.astro_group_attn_fwd(cache, a["q"], k, v, 2, group, a["out"], a["lse"], ws, stream=stream)
        if group == 1:
            for call in (lambda x: A.astro_chunk_attn_fwd(cache, q, k, v, 2, out, x, ws, stream=stream),
                         lambda x: A.astro_chunk_attn_bwd(cache, q, k, v, out, x, do, 2, *g, ws, stream=stream),
                         lambda x: A.astro_chunk_attn_bwd_full(cache, q, k, v, out, x, do, 2, *g, *ring, ws, stream=stream)):
                for x in (lse.flatten()[1:], lse.half(), lse.transpose(1, 2)):
                    with pytest.raises(ValueError):
                        call(x)
        with pytest.raises(A.AstroError) as e:
            A.astro_group_attn_fwd(cache, q, k, v, 2, group, out, lse, ws[:256], stream=stream)
        assert e.value.code == binding.ASTRO_ERR_WORKSPACE
        # a subclass of Tensor still goes through
        A.astro_group_attn_fwd(cache, q.as_subclass(type("Sub", (torch.Tensor,), {})), k, v, 2, group, out, lse, ws, stream=stream)
        assert torch.equal(out, results[-1][0])
        # what both refuse, an error of the library and a subclass
        assert [a for *_, a in answers[len(took):]] == ([None] * (14 if group == 1 else 5) + [binding.ASTRO_ERR_WORKSPACE, None] if stream is None else [])
        cache.close()
        with pytest.raises(A.AstroError):
            A.astro_kvcache_append(cache, k0, v0, 2, stream=stream)
        del answers[:]
    for a, b in zip(*results):
        assert torch.equal(a, b)


@pytest.mark.gpu
def test_loss_gives_what_the_ctypes_path_gives_on_the_current_stream(answers):
    gen = torch.Generator("cuda:0").manual_seed(5)
    x = [torch.randn((3, 5, 104), generator=gen, device="cuda:0").bfloat16() for _ in range(4)]
    adv, mask = torch.randn(3, generator=gen, device="cuda:0"), torch.tensor([0, 1, 1], dtype=torch.int32, device="cuda:0")
    ws = torch.empty(A.astro_nft_loss_workspace_bytes(3, 520), dtype=torch.uint8, device="cuda:0")
    side, results = torch.cuda.Stream(), []
    for stream, a_max in ((None, 1.0), (side, 1.0), (None, 1)):  # an int goes through ctypes
        loss, grad = torch.full((3,), -1.0, device="cuda:0"), torch.full(x[0].shape, -1.0, device="cuda:0")
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            A.astro_nft_loss(*x, adv, mask, a_max, 0.9, 0.1, loss, grad, ws, stream=stream)
        side.synchronize()
        results.append((loss, grad))
    assert answers == [("loss", 12, 0), ("loss", 12, None)]  # the call with an int is not taken
    for r in results[1:]:
        assert torch.equal(r[0], results[0][0]) and torch.equal(r[1], results[0][1])
    for change in (dict(old=x[1].float()), dict(adv=adv[:1].expand(3)), dict(mask=mask.repeat(2)[::2]), dict(loss=loss.repeat(2)[::2]),
                   dict(grad=grad.transpose(0, 1))):
        a = dict(old=x[1], adv=adv, mask=mask, loss=loss, grad=grad)
        a.update(change)
        with pytest.raises(ValueError):
            A.astro_nft_loss(x[0], a["old"], x[2], x[3], a["adv"], a["mask"], 1.0, 0.9, 0.1, a["loss"], a["grad"], ws)


ALONE = """
import sys, warnings
sys.path.insert(0, {root!r})
import torch
if {other!r}:
    torch.version.git_version = "another"
with warnings.catch_warnings(record=True) as told:
    warnings.simplefilter("always")
    import paper_2603_17051_amd as A
assert A.__file__.startswith({root!r})
assert any("ctypes" in str(w.message) for w in told), told
c = A.astro_kvcache_create(2, 2, 64, 4, 8, 4, 1, 2, (12, 10, 10), host_only=True)
A.astro_kvcache_append(c, n_frames=2)
assert A.astro_kvcache_tables(c)[2] == [2, 2]
x = torch.zeros(2, 32, 2, 64, dtype=torch.bfloat16)
try:
    A.astro_chunk_attn_fwd(c, x, x, x, 1, torch.zeros(1), torch.zeros(1), torch.zeros(1))
except ValueError as e:
    assert "device tensor" in str(e)
else:
    raise SystemExit("a host tensor was taken")
"""


@pytest.mark.parametrize("other", [False, True])
def test_a_module_that_is_missing_or_of_another_torch_leaves_all_calls_to_ctypes(other, tmp_path):
    package = os.path.dirname(binding.__file__)
    copy = tmp_path / "paper_2603_17051_amd"
    copy.mkdir()
    for name in os.listdir(package):
        if name.endswith(".py") or name == "libastro.so" or (other and name == os.path.basename(build.NATIVE_PATH)):
            shutil.copy(os.path.join(package, name), copy)
    r = subprocess.run([sys.executable, "-c", ALONE.format(root=str(tmp_path), other=other)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr


def test_the_module_is_the_one_of_this_python_and_torch():
    assert binding._native.__file__ == build.NATIVE_PATH and build.NATIVE_PATH.endswith(sysconfig.get_config_var("EXT_SUFFIX"))
    assert binding._native.built_for_torch.startswith(torch.__version__)


class OnDevice:
    """What the binding's checks see of a contiguous device tensor."""
    is_cuda = True

    def __init__(self, dtype, *shape, dense=True):
        self.dtype, self.shape, self.is_contiguous, self.device = dtype, shape, lambda: dense, "cuda:0"

    def numel(self):
        return math.prod(self.shape)

    def element_size(self):
        return 2 if self.dtype is torch.bfloat16 else 4

    def data_ptr(self):
        return 1 << 20


@pytest.mark.parametrize("lse,fits", [
    (OnDevice(torch.float32, 2, 2, 32), True), (OnDevice(torch.float32, 200), True), (OnDevice(torch.float32, 127), False),
    (OnDevice(torch.bfloat16, 2, 2, 32), False), (OnDevice(torch.float32, 2, 2, 32, dense=False), False)])
def test_log_sum_exps_of_the_calls_without_candidates_have_room(lse, fits, monkeypatch):
    """(a host-only handle answers the C ABI's calls with a state error: nothing is launched)"""
    monkeypatch.setattr(binding, "_stream", lambda stream: ctypes.c_void_p(None))
    cache = A.astro_kvcache_create(host_only=True, **GOOD)
    x, ws = OnDevice(torch.bfloat16, 2, 32, 2, 64), OnDevice(torch.float32, 1 << 16)
    g, ring = [OnDevice(torch.float32, 2, 32, 2, 64)] * 3, [OnDevice(torch.float32, 2, 128, 2, 64)] * 2
    for call in (lambda: A.astro_chunk_attn_fwd(cache, x, x, x, 1, x, lse, ws),
                 lambda: A.astro_chunk_attn_bwd(cache, x, x, x, x, lse, x, 1, *g, ws),
                 lambda: A.astro_chunk_attn_bwd_full(cache, x, x, x, x, lse, x, 1, *g, *ring, ws)):
        with pytest.raises(A.AstroError if fits else ValueError):
            call()
    cache.close()


def test_the_loss_takes_its_small_arguments_and_outputs_dense_only(monkeypatch):
    """The kernels read and write them one after another from their addresses, whatever their strides."""
    took = []
    for name in ("astro_nft_loss", "astro_nft_loss_static"):
        monkeypatch.setattr(binding._lib, name, lambda *args: took.append(args) or 0)
    monkeypatch.setattr(binding, "_stream", lambda stream: ctypes.c_void_p(None))
    x, ws = OnDevice(torch.bfloat16, 3, 8), OnDevice(torch.float32, 1 << 16)
    for strided in (None, 0, 1, 2, 3):
        adv, mask, loss, grad = (OnDevice(t, *shape, dense=i != strided) for i, (t, shape) in enumerate(
            [(torch.float32, (3,)), (torch.int32, (3,)), (torch.float32, (3,)), (torch.float32, (3, 8))]))
        for call in (lambda: A.astro_nft_loss(x, x, x, x, adv, mask, 1.0, 1.0, 0.1, loss, grad, ws),
                     lambda: A.astro_nft_loss_static(x, x, x, x, adv, mask, 1.0, 1.0, 0.1, loss, grad)):
            del took[:]
            if strided is None:
                call()
                assert len(took) == 1
            else:
                with pytest.raises(ValueError):
                    call()
                assert not took


def test_memory_that_kernels_cannot_reach_is_refused(monkeypatch):
    """Log-sum-exps, workspaces and everything of the loss, whose kernels would have been given host addresses."""
    took = []
    for name in ("astro_nft_loss", "astro_nft_loss_static"):
        monkeypatch.setattr(binding._lib, name, lambda *args: took.append(args) or 0)
    monkeypatch.setattr(binding, "_stream", lambda stream: ctypes.c_void_p(None))
    cache = A.astro_kvcache_create(host_only=True, **GOOD)
    x, ws, lse = OnDevice(torch.bfloat16, 2, 32, 2, 64), OnDevice(torch.float32, 1 << 16), OnDevice(torch.float32, 2, 2, 32)
    g, ring = [OnDevice(torch.float32, 2, 32, 2, 64)] * 3, [OnDevice(torch.float32, 2, 128, 2, 64)] * 2
    for l, w in [(torch.zeros(2, 2, 32), ws), (lse, torch.zeros(1 << 16))]:
        for call in (lambda: A.astro_chunk_attn_fwd(cache, x, x, x, 1, x, l, w),
                     lambda: A.astro_group_attn_fwd(cache, x, x, x, 1, 1, x, l, w),
                     lambda: A.astro_chunk_attn_bwd(cache, x, x, x, x, l, x, 1, *g, w),
                     lambda: A.astro_group_attn_bwd(cache, x, x, x, x, l, x, 1, 1, *g, w),
                     lambda: A.astro_chunk_attn_bwd_full(cache, x, x, x, x, l, x, 1, *g, *ring, w)):
            with pytest.raises(ValueError, match="device tensor"):
                call()
    cache.close()
    elems, n = OnDevice(torch.bfloat16, 3, 8), OnDevice(torch.float32, 3)
    good = [elems] * 4 + [n, OnDevice(torch.int32, 3), n, OnDevice(torch.float32, 3, 8), ws]
    for i, t in enumerate(good):
        a = list(good)
        a[i] = torch.zeros(t.shape, dtype=t.dtype)
        for call, args in ((A.astro_nft_loss, a), (A.astro_nft_loss_static, a[:8])):
            if i < len(args):
                with pytest.raises(ValueError, match="device tensor"):
                    call(*args[:6], 1.0, 1.0, 0.1, *args[6:])
    assert not took
    with pytest.raises(ValueError, match="device tensor"):
        A.astro_calib_copy(torch.zeros(4), torch.zeros(4))
    with pytest.raises(ValueError, match="device tensor"):
        A.astro_calib_mfma(torch.zeros(8 * 256 * 4), 1, 1, torch.zeros(256))
