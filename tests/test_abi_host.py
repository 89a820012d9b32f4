"""CPU-side checks of the C-ABI library: it loads, exports every symbol the header declares, and the
host-only logic (configuration validation, band sizes) behaves.  No kernel is launched here."""
import ctypes as C
import os
import re

import numpy as np
import pytest

import paper_2605_09490_amd as tkv
from paper_2605_09490_amd import binding
from oracle import tkv_oracle as O

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared_symbols():
    src = open(os.path.join(ROOT, "include", "tkv.h")).read()
    src = re.sub(r"/\*.*?\*/", "", src, flags=re.S)
    return sorted(set(re.findall(r"\b(tkv_[a-z0-9_]+)\s*\(", src)))


def test_library_exports_every_declared_symbol():
    lib = tkv.load_library()
    names = _declared_symbols()
    assert "tkv_create" in names and "tkv_attend_and_score" in names and "tkv_migrate" in names
    for n in names:
        assert hasattr(lib, n), n
    assert sorted(binding.SYMBOLS) == names


def test_config_struct_matches_header_field_order():
    src = open(os.path.join(ROOT, "include", "tkv.h")).read()
    body = src[src.index("typedef struct {", src.index("tkv_prefetch_mode;")):]
    body = body[:body.index("} tkv_config;")]
    body = re.sub(r"/\*.*?\*/", "", body, flags=re.S)
    fields = []
    for decl in body.split(";"):
        decl = decl.strip().replace("typedef struct {", "")
        if not decl:
            continue
        m = re.match(r"(?:void\*?|void)\s*\(\*(\w+)\)", decl)
        if m:
            fields.append(m.group(1))
            continue
        names = decl.split(None, 1)[1] if " " in decl else ""
        fields += [n.strip().lstrip("*") for n in names.split(",")]
    assert fields == [f[0] for f in binding.tkv_config._fields_]


def test_create_rejects_bad_configs_before_touching_the_device():
    lib = tkv.load_library()

    def status(**kw):
        cfg = binding.tkv_config()
        base = dict(n_layers=1, batch=1, n_q_heads=8, n_kv_heads=2, head_dim=64, max_tokens=64, kv_dtype=0, t2_format=0)
        base.update(kw)
        for k, v in base.items():
            setattr(cfg, k, v)
        h = C.c_void_p()
        st = lib.tkv_create(C.byref(cfg), C.byref(h))
        assert not h.value
        return st

    assert status(head_dim=96) == tkv.TKV_EINVAL
    assert status(n_q_heads=7) == tkv.TKV_EINVAL
    assert status(n_q_heads=18, n_kv_heads=2) == tkv.TKV_EINVAL      # group of 9
    assert status(max_tokens=0) == tkv.TKV_EINVAL
    assert status(max_tokens=1 << 24) == tkv.TKV_EINVAL
    assert status(kv_dtype=7) == tkv.TKV_EINVAL
    assert status(t2_format=2) == tkv.TKV_EINVAL
    assert status(k_window=-1) == tkv.TKV_EINVAL
    assert status(prefetch_mode=5) == tkv.TKV_EINVAL
    assert status(scorer=4) == tkv.TKV_EINVAL
    assert status(scorer=2, redundancy_weight=-1.0) == tkv.TKV_EINVAL
    assert lib.tkv_create(None, None) == tkv.TKV_EINVAL
    assert b"tkv_create" in lib.tkv_last_error(None)
    lib.tkv_destroy(None)


def test_tier_counts_agree_with_oracle_and_reject_bad_policy():
    rng = np.random.default_rng(0)
    for _ in range(200):
        m = int(rng.integers(0, 40000))
        cut = np.sort(rng.integers(0, 10 ** 6 + 1, size=3))
        pol = (int(cut[0]), int(cut[1] - cut[0]), int(cut[2] - cut[1]), int(10 ** 6 - cut[2]))
        ev = int(rng.integers(0, m + 1)) if rng.random() < 0.3 else 0
        assert tkv.tier_counts(pol, m, ev) == O.tier_counts(m, pol, ev)
        assert tkv.tier_counts(pol, m, ev, count_rule=1) == O.tier_counts_alg1(m, pol, ev)
    with pytest.raises(tkv.TkvError):
        tkv.tier_counts((1, 2, 3, 4), 10)
    with pytest.raises(tkv.TkvError):
        tkv.tier_counts((250000, 250000, 250000, 250000), 10, 0, count_rule=5)


def test_host_code_under_sanitizers_host_only_part():
    """The library's host code built with AddressSanitizer and UndefinedBehaviorSanitizer (host side only) and driven by
    tests/native/host_sanitize_check.cpp: here the part that needs no GPU (configuration validation, band sizes, NULL
    handles).  The full scenario runs in the GPU suite."""
    import subprocess
    from paper_2605_09490_amd import build
    exe = build.HOST_CHECK
    if not os.path.exists(exe):
        build.build_host_check()
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:protect_shadow_gap=0", UBSAN_OPTIONS="halt_on_error=1")
    r = subprocess.run([exe, "--host-only"], capture_output=True, text=True, timeout=120, env=env)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "host sanitizer check passed" in r.stdout


def test_sources_compile_without_warnings():
    """Every unit of the library, host and device side, front end only: an index past the end of an array in a template
    instantiation, for one, is a warning that an optimised build goes along with."""
    import subprocess
    from concurrent.futures import ThreadPoolExecutor
    from paper_2605_09490_amd import build

    def check(unit):
        src, extra, _ = unit
        r = subprocess.run([build._hipcc(), *build.FLAGS, *extra, "-fsyntax-only", "-Wno-unused-command-line-argument",
                            os.path.join(build.CSRC, src)], capture_output=True, text=True, timeout=600)
        return build.diagnostics(r.stderr) if r.returncode == 0 else r.stderr

    with ThreadPoolExecutor(max_workers=4) as ex:
        said = [d for d in ex.map(check, build.UNITS) if d]
    assert not said, said[0][:2000]


@pytest.mark.parametrize("scenario", ["refused_allocations", "allocations_before_use", "route_follows_from_the_shape",
                                      "parts_of_pairs", "few_heads_on_the_vector_alus", "long_lists_fill_the_chip", "chunk_splits", "chunk_tokens_per_launch", "kernel_times"])
def test_host_code_on_a_runtime_that_launches_nothing(scenario):
    """tests/native/fake_runtime_check.cpp: the host code against a stand-in for the HIP runtime; allocations can be refused,
    and every launch is compared with the memory alive."""
    import subprocess
    from paper_2605_09490_amd import build
    r = subprocess.run([build.build_fake_check(), scenario], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and f"{scenario}: ok" in r.stdout, r.stdout + r.stderr


def test_launches_that_the_gpu_tests_mean():
    """Shapes of tests/test_gpu_shapes.py that are there for what a launch does with them: pairs in so many parts, whole pairs whose
    logits do not fit the LDS.  Both follow from rules on the shape, which may move."""
    import re
    import subprocess

    import test_gpu_shapes as shapes
    from paper_2605_09490_amd import build
    exe = build.build_fake_check()

    def route(s):
        tokens = s["context"] + s.get("decode_steps", 4)
        args = [str(s[k]) for k in ("n_layers", "batch", "n_q_heads", "n_kv_heads", "head_dim")] + [str(tokens)]
        r = subprocess.run([exe, "route", *args], capture_output=True, text=True, timeout=60)
        assert r.returncode == 0, r.stdout + r.stderr
        return [int(x) for x in re.fullmatch(r"step (\d+) whole (\d+) in (\d+) parts; call (\d+) whole; lds (\d+)\n", r.stdout).groups()]

    seen = set()
    for n, pairs, _, _, s in shapes.STEPS_IN_PARTS:
        whole, in_parts, parts, _, _ = route(s)
        assert (parts, in_parts) == (n, pairs), (s, whole, in_parts, parts)
        seen.add(parts)
    assert seen == set(range(2, 9))
    for s in shapes.STEPS_BEYOND_THE_LDS:
        whole, _, _, _, lds = route(s)
        assert whole > 0 and s["context"] > lds, (s, whole, lds)
    for s in shapes.CALLS_BEYOND_THE_LDS:
        _, _, _, whole, lds = route(dict(s, n_layers=1))
        assert whole > 0 and s["context"] > lds, (s, whole, lds)
    whole, in_parts, _, call, _ = route(shapes.PRECISION)
    assert whole > 0 and in_parts == 0 and call == 0


def test_current_stream_without_the_raw_handle(monkeypatch):
    """The function that gives a stream's raw handle is a private one of torch's: without it the public way is taken."""
    import importlib.util
    import types

    import torch
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda device=None: types.SimpleNamespace(cuda_stream=40 + device))
    spec = importlib.util.spec_from_file_location("binding_of_its_own", binding.__file__)
    own = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(own)
    assert own.TieredKV._stream(None) == 43
    assert own.TieredKV._stream(types.SimpleNamespace(cuda_stream=7)) == 7


def test_chunk_scratch_comes_from_the_calls_own_stream(monkeypatch):
    """PyTorch's allocator keeps a pool per stream.  The scratch of a handle's first chunk is written on the stream that the
    call names, so it has to come from that stream's pool, not from the one of whatever stream is current."""
    import contextlib
    import types

    import torch
    taken, current = [], [None]

    @contextlib.contextmanager
    def on_stream(s):
        before, current[0] = current[0], s or current[0]
        yield
        current[0] = before

    def create(cfg, h):
        lib.dev_alloc = cfg._obj.dev_alloc
        lib.dev_alloc(64, None)
        return tkv.TKV_OK

    def chunk(*_):
        lib.dev_alloc(64, None)
        return tkv.TKV_OK

    lib = types.SimpleNamespace(tkv_create=create, tkv_attend_and_score_chunk=chunk, tkv_destroy=lambda h: None)
    empty = torch.empty
    monkeypatch.setattr(binding, "load_library", lambda: lib)
    monkeypatch.setattr(torch.cuda, "stream", on_stream)
    monkeypatch.setattr(torch, "empty", lambda *a, **kw: (taken.append(current[0]), empty(64, dtype=torch.uint8))[1])
    monkeypatch.setattr(tkv.TieredKV, "_dev_tensor", lambda self, t, shape, dtype=None: None)
    kv = tkv.TieredKV(1, 1, 4, 2, 64, 128)
    side = types.SimpleNamespace(cuda_stream=7)
    kv.attend_and_score_chunk(0, np.zeros((1, 2)), out=np.zeros(1), stream=side)
    assert taken == [None, side]
