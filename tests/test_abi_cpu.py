"""Host-only checks of the C ABI: the library loads, exports every function that
include/mbp.h declares, validates configurations, and agrees with the seeded
generator's weight manifest.  No compute call is made (no GPU here)."""
import ctypes
import os
import re

import pytest

import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def mbp():
    import paper_2608_15454_amd as m

    if not os.path.exists(m.lib_path()):
        pytest.fail("libmbp.so is not built; run __graft_entry__.build()")
    m.lib()
    return m


def _declared_functions():
    text = open(os.path.join(ROOT, "include", "mbp.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(mbp_[a-z_]+)\s*\(", text)))


def test_header_declares_the_four_entry_points():
    names = _declared_functions()
    for n in ("mbp_init", "mbp_prefill", "mbp_decode_step", "mbp_accept"):
        assert n in names


def test_library_exports_every_declared_symbol(mbp):
    L = ctypes.CDLL(mbp.lib_path())
    missing = [n for n in _declared_functions() if not hasattr(L, n)]
    assert not missing, missing


def _cfg(mbp, wl="lca_d1024_b1", **kw):
    w = synth.WORKLOADS[wl]
    args = dict(max_batch=w.batch, max_ctx=w.prompt_len + w.gen_len + 8, max_n=8)
    args.update(kw)
    return mbp.make_config(w.model, **args)


def test_manifest_of_models_without_mb_head(mbp):
    for model in (synth.TINY_FXT, synth.D1024_FXT):
        cfg = mbp.make_config(model, max_batch=1, max_ctx=512, max_n=8)
        lib_man = mbp.weight_manifest(cfg)
        gen_man = synth.manifest(model)
        assert [n for n, _ in lib_man] == [n for n, _ in gen_man]
        assert mbp.lib().mbp_workspace_bytes(ctypes.byref(cfg)) > 0


@pytest.mark.parametrize("wl", list(synth.WORKLOADS))
def test_manifest_matches_generator(mbp, wl):
    cfg = _cfg(mbp, wl)
    lib_man = mbp.weight_manifest(cfg)
    gen_man = synth.manifest(synth.WORKLOADS[wl].model)
    assert len(lib_man) == len(gen_man)
    for (ln, (r, c)), (gn, shape) in zip(lib_man, gen_man):
        assert ln == gn
        assert r * c == int(__import__("numpy").prod(shape))
        assert (r, c) == (shape[0], shape[1] if len(shape) > 1 else 1)


def test_workspace_bytes_positive_and_monotone(mbp):
    L = mbp.lib()
    a = L.mbp_workspace_bytes(ctypes.byref(_cfg(mbp, max_ctx=1000)))
    b = L.mbp_workspace_bytes(ctypes.byref(_cfg(mbp, max_ctx=2000)))
    assert 0 < a < b


@pytest.mark.parametrize("field,value", [
    ("d_model", 0), ("n_heads", 3), ("d_ff", 100), ("n_lm", -1), ("head", 5), ("dtype", 7),
    ("max_batch", 0), ("max_ctx", 1), ("max_n", 0), ("max_n", 9), ("max_patch", -1),
    ("window_mode", 2), ("rope_base", 0.0),
])
def test_invalid_configs_rejected(mbp, field, value):
    L = mbp.lib()
    cfg = _cfg(mbp)
    setattr(cfg, field, value)
    assert L.mbp_workspace_bytes(ctypes.byref(cfg)) == 0
    assert L.mbp_weight_count(ctypes.byref(cfg)) == mbp.EINVAL
    h = ctypes.c_void_p()
    ptrs = (ctypes.c_void_p * 1)(1)
    assert L.mbp_init(ctypes.byref(cfg), ptrs, 1, ctypes.c_void_p(256), 1 << 40, None, ctypes.byref(h)) == mbp.EINVAL
    assert not h.value


def test_window_mode_1_accepted(mbp):
    """Window mode 1 keeps MB rows for the whole sequence: accepted with the pure space
    rule and no max_window, with a larger workspace than mode 0."""
    L = mbp.lib()
    cfg = _cfg(mbp)
    a = L.mbp_workspace_bytes(ctypes.byref(cfg))
    cfg.window_mode = 1
    b = L.mbp_workspace_bytes(ctypes.byref(cfg))
    cfg.max_patch = 0
    c = L.mbp_workspace_bytes(ctypes.byref(cfg))
    assert 0 < a < b and c > 0


def test_pure_space_rule_needs_max_window(mbp):
    L = mbp.lib()
    model = synth.WORKLOADS["tiny_f32"].model.replace(max_patch=0)
    cfg = mbp.make_config(model, max_batch=1, max_ctx=100, max_n=4)
    assert L.mbp_workspace_bytes(ctypes.byref(cfg)) == 0
    cfg.max_window = 64
    assert L.mbp_workspace_bytes(ctypes.byref(cfg)) > 0


def test_init_argument_checks_before_any_device_work(mbp):
    L = mbp.lib()
    cfg = _cfg(mbp, "tiny_f32")
    n = L.mbp_weight_count(ctypes.byref(cfg))
    ptrs = (ctypes.c_void_p * n)(*([4096] * n))
    h = ctypes.c_void_p()
    ws = L.mbp_workspace_bytes(ctypes.byref(cfg))
    # wrong weight count, null weight, misaligned workspace, small workspace, null out
    assert L.mbp_init(ctypes.byref(cfg), ptrs, n - 1, ctypes.c_void_p(4096), ws, None, ctypes.byref(h)) == mbp.EINVAL
    ptrs0 = (ctypes.c_void_p * n)(*([4096] * (n - 1) + [0]))
    assert L.mbp_init(ctypes.byref(cfg), ptrs0, n, ctypes.c_void_p(4096), ws, None, ctypes.byref(h)) == mbp.EINVAL
    assert L.mbp_init(ctypes.byref(cfg), ptrs, n, ctypes.c_void_p(4096 + 8), ws, None, ctypes.byref(h)) == mbp.EINVAL
    assert L.mbp_init(ctypes.byref(cfg), ptrs, n, ctypes.c_void_p(4096), ws - 1, None, ctypes.byref(h)) == mbp.ECAPACITY
    assert L.mbp_init(ctypes.byref(cfg), ptrs, n, ctypes.c_void_p(4096), ws, None, None) == mbp.EINVAL


def test_null_handle_calls(mbp):
    L = mbp.lib()
    assert L.mbp_prefill(None, None, None, 1) == mbp.EINVAL
    assert L.mbp_decode_step(None, 3, 0.5, 0, None, None, None) == mbp.EINVAL
    assert L.mbp_accept(None, None, None) == mbp.EINVAL
    assert L.mbp_reset(None) == mbp.EINVAL
    assert L.mbp_row_length(None, 0) == mbp.EINVAL
    L.mbp_destroy(None)


def test_kernels_use_no_scratch_memory(mbp):
    """Every kernel keeps its working state in registers and LDS.  Scratch memory inside
    a hot loop costs a multiple of the kernel's time: an accumulator array that the
    compiler indexed at run time, and so placed in scratch, made the tiled GEMM three
    times slower with no error.  The build records each kernel's resources from the
    compiler's remarks.  Allowed, measured: the d=2048 engine's multi-row and split
    variants, which spill a few dwords at the 256-VGPR limit (the d=2048 verification
    workload launches the engine twice per run; its decode steps run on the per-kernel
    path)."""
    path = os.path.join(ROOT, "paper_2608_15454_amd", "_build", "kernel_resources.tsv")
    assert os.path.exists(path), "rebuild: the build writes _build/kernel_resources.tsv"
    rows = [line.rstrip("\n").split("\t") for line in open(path)][1:]
    assert len(rows) > 50 and {r[0] for r in rows} >= {"kernels.hip", "planes.hip", "engine.hip"}
    bad = []
    for src, name, _vgprs, _agprs, scratch, _occ, _lds in rows:
        if int(scratch) == 0 or (src == "engine.hip" and "Li2048E" in name and int(scratch) <= 64):
            continue
        bad.append((src, name, int(scratch)))
    assert not bad, bad


def test_counter_records_follow_code_not_comments(tmp_path):
    """A counter record stays valid across edits to comments and layout, and only
    those: bench.py compares a digest of the source's code."""
    import bench

    base = "int f(int a) {\n  return a + 1;  // one more\n}\n/* note */\n"
    cases = {
        "comment": "int f(int a) {\n  return a + 1;  // one more than a\n}\n/* another note */\n",
        "layout": "int f(int a)\n{\n    return a + 1;\n}\n",
        "code": "int f(int a) {\n  return a + 2;  // one more\n}\n/* note */\n",
    }
    p0 = tmp_path / "base.hip"
    p0.write_text(base)
    d0 = bench.code_digest(str(p0))
    for name, text in cases.items():
        p = tmp_path / f"{name}.hip"
        p.write_text(text)
        assert (bench.code_digest(str(p)) == d0) == (name != "code"), name
    # every record in profiles/ names a code digest
    for rec in os.listdir(os.path.join(ROOT, "profiles")):
        if rec.endswith("_hbm_counters.md"):
            assert "code sha256: `" in open(os.path.join(ROOT, "profiles", rec)).read(), rec


@pytest.mark.parametrize("cls,edited,valid", [("gemm", "planes.hip", False), ("gemm", "kernels.hip", False), ("gemm", "dev.h", False),
                                              ("gemm", "engine.hip", True), ("engine", "engine.hip", False), ("engine", "planes.hip", True),
                                              ("attention", "kernels.hip", False), ("attention", "planes.hip", True)])
def test_counter_records_follow_every_source(tmp_path, cls, edited, valid):
    """A record of a class counts while no source of that class's kernels has changed."""
    import bench

    for f in ("kernels.hip", "planes.hip", "engine.hip", "dev.h"):
        (tmp_path / f).write_text(f"int f() {{ return {len(f)}; }}\n")
    rec = [f"- class: {cls}", "- workload: w", "- hbm bytes per launch: 12"] + bench.digest_lines(cls, str(tmp_path))
    (tmp_path / f"{cls}_w_hbm_counters.md").write_text("\n".join(rec) + "\n")
    assert bench.measured_traffic(cls, "w", str(tmp_path), str(tmp_path)) == 12
    (tmp_path / edited).write_text("int f() { return 0; }\n")
    assert bench.measured_traffic(cls, "w", str(tmp_path), str(tmp_path)) == (12 if valid else None)


def test_inline_asm_declares_m0():
    """An asm statement that writes m0 lists it as clobbered: the compiler keeps lane and
    LDS indices there and would read the asm's value."""
    import re

    seen = 0
    for f in sorted(os.listdir(os.path.join(ROOT, "paper_2608_15454_amd", "csrc"))):
        src = open(os.path.join(ROOT, "paper_2608_15454_amd", "csrc", f)).read()
        for stmt in re.findall(r"\basm\s+volatile\s*\((.*?)\);", src, flags=re.S):
            if "m0," in stmt.split("::")[0]:
                seen += 1
                assert '"m0"' in stmt.rsplit(":", 1)[1], (f, stmt)
    assert seen
