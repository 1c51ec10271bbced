"""The C ABI without a GPU: the library loads, exports every symbol the header
declares, and rejects malformed tables / arguments on the host."""
import ctypes as C
import os
import re
import shutil
import subprocess
import sys
import sysconfig
import types

import numpy as np
import pytest
import torch

import paper_2509_25041_amd as grace
from paper_2509_25041_amd import binding
from workloads import CONFIGS, make_workload

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_symbols():
    text = open(os.path.join(ROOT, "include", "grace_moe.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(grace_[a-z_]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    lib = grace.load_library()
    names = declared_symbols()
    assert set(names) == set(binding.EXPORTS)
    for n in names:
        assert getattr(lib, n) is not None
    assert os.path.dirname(grace.library_path()).endswith("paper_2509_25041_amd")


def test_asking_for_the_stream_initialises_the_device(monkeypatch):
    """GraceTable may be the first GPU call of a process: torch's own initialisation, and its messages where it is not
    possible, come before the library's."""
    if torch.cuda.is_initialized():
        pytest.skip("the device is in use already")

    def lazy_init():
        raise RuntimeError("initialised here")

    monkeypatch.setattr(torch.cuda, "_lazy_init", lazy_init)
    with pytest.raises(RuntimeError, match="initialised here"):
        grace.GraceTable(1, 1, 1, [0], [1], [0, 1], [0])


def test_binding_has_the_entry_points_under_their_own_names():
    """Every exported call is reachable from Python under the C name (functions of the binding, re-exported
    by the package), the table's calls as methods of GraceTable."""
    methods = {"grace_table_create": "__init__", "grace_table_destroy": "destroy", "grace_table_info": "__init__",
               "grace_table_instances": "instances", "grace_table_local_experts": "local_experts",
               "grace_table_set_fold_limits": "set_fold_limits"}
    for n in binding.EXPORTS:
        if n in methods:
            assert callable(getattr(grace.GraceTable, methods[n]))
        else:
            assert callable(getattr(binding, n)), n
            assert getattr(grace, n) is getattr(binding, n), n


def test_valid_tables_pass_validation():
    for cfg in CONFIGS.values():
        pl = make_workload(cfg, T=256).placement
        grace.grace_table_validate(pl.E, pl.R, pl.N, pl.rank_node, pl.poll_weight, pl.inst_ptr, pl.inst_rank)


GOOD = dict(E=2, R=2, N=1, rank_node=[0, 0], poll_weight=[1, 2], inst_ptr=[0, 1, 3], inst_rank=[0, 0, 1])


@pytest.mark.parametrize("patch,status", [
    (dict(poll_weight=[1, 0]), -3),                 # zero weight
    (dict(poll_weight=[1, 70000]), -3),             # oversized weight
    (dict(inst_ptr=[0, 0, 2], inst_rank=[0, 1, 1]), -3),   # expert without instance
    (dict(inst_rank=[0, 0, 2]), -3),                # rank out of range
    (dict(inst_rank=[0, 1, 1]), -3),                # duplicate (expert, rank)
    (dict(inst_rank=[0, 1, 0]), -3),                # unsorted ranks
    (dict(rank_node=[1, 0], N=2), -3),              # decreasing rank_node
    (dict(rank_node=[0, 1]), -3),                   # node id out of range
    (dict(inst_ptr=[1, 2, 3]), -3),                 # inst_ptr not starting at 0
    (dict(E=0), -1),
    (dict(E=300, inst_ptr=list(range(301)), inst_rank=[0] * 300), -2),
])
def test_malformed_tables_are_rejected(patch, status):
    a = {**GOOD, **patch}
    with pytest.raises(grace.GraceError) as ei:
        grace.grace_table_validate(a["E"], a["R"], a["N"], a["rank_node"], a["poll_weight"], a["inst_ptr"],
                                   a["inst_rank"])
    assert ei.value.status == status
    assert grace.grace_last_error() != ""


def test_null_and_range_checks_without_device():
    lib = grace.load_library()
    assert lib.grace_table_validate(2, 2, 1, None, None, None, None) == -1
    assert lib.grace_table_destroy(None) == 0
    assert lib.grace_table_info(None, None, None, None, None, None) == -1
    # compute entry points refuse a null table before touching the device
    assert lib.grace_route(None, 0, 0, None, 1, 1, 1, 1, None, None, None, None, None, None, None, None) == -1
    assert lib.grace_permute(None, None, 1, 1, None, 8, 1, None, None, None, None, None, None, None, None) == -1
    assert lib.grace_expert_ffn(None, 0, None, None, 1, 1, 8, 8, 1, None, None, None, None, None, None) == -1
    assert lib.grace_shared_ffn(None, 1, 8, 8, 0, 1, None, None, None, None, None, None) == -1
    assert lib.grace_shared_ffn(None, 1, 12, 8, 1, 1, None, None, None, None, None, None) == -2   # bf16 needs d % 8 == 0
    assert lib.grace_combine(None, None, None, 1, 1, 3, 1, None, None, None) == -2               # 6-byte rows
    assert lib.grace_combine(None, None, None, 1, 1, 8, 1, None, None, None) == -1               # null pointers
    assert lib.grace_combine(None, None, None, 0, 1, 8, 1, None, None, None) == 0                # nothing to do
    assert lib.grace_combine_share(None, None, None, 1, 1, 3, 1, None, None, None, None) == -2
    assert lib.grace_combine_share(1 << 20, 1 << 20, 1 << 20, 1, 1, 8, 1, None, None, 1 << 20, None) == -1     # no state
    assert lib.grace_mfma_sustained(1, 1, None, None) == -1
    assert lib.grace_table_set_fold_limits(None, -1, -1) == -1
    assert lib.grace_permute_rows(None, None, 1, 1, 8, 1, None, None) == -1
    assert lib.grace_shared_ffn_up_scatter(None, 1, 8, 8, 1, 1, None, None, None, None, 0, None, None) == -1
    assert lib.grace_permute_rows(None, None, 0, 1, 8, 1, None, None) == 0
    assert lib.grace_route_permute_static(None, 0, 0, None, 1, 1, 1, 1, None, None, None, None, None, None, None, 8, 1, None,
                                          None, None, None, None, None, None) == -1
    assert lib.grace_expert_ffn_up_share(None, 0, None, None, 1, 1, 8, 8, 1, None, None, None, None, None) == -1
    assert lib.grace_expert_ffn_down_share(None, 0, None, 1, 1, 8, 8, 1, None, None, None, None, None) == -1
    assert lib.grace_expert_ffn_down_fresh(None, 0, None, 1, 1, 8, 8, 1, None, None, None, None) == -1
    assert lib.grace_send_lists(None, 0, None, 1, 1, None, None, None, None, None, None, None, None) == -1


def test_workspace_bytes():
    assert grace.grace_workspace_bytes(-1, 8, 2, 11) == 0
    small = grace.grace_workspace_bytes(256, 8, 2, 11)
    assert small >= 2 * 4 * 8 * 4
    big = grace.grace_workspace_bytes(4096, 64, 8, 76, 2048, 1024, 0, grace.GRACE_BF16)
    assert big >= 4096 * 8 * 1024 * 2
    assert grace.grace_workspace_bytes(4096, 64, 8, 76, 2048, 1024, 0, grace.GRACE_F32) >= 2 * (big - 256)


@pytest.mark.parametrize("E,k,I,f,dt", [
    (64, 8, 76, 1024, grace.GRACE_BF16), (64, 8, 76, 1024, grace.GRACE_F32), (128, 8, 150, 768, grace.GRACE_BF16), (60, 4, 69, 1408, grace.GRACE_BF16),
    (8, 2, 11, 14336, grace.GRACE_BF16), (12, 9, 12, 7400, grace.GRACE_BF16), (200, 1, 255, 2048, grace.GRACE_F32), (64, 64, 300, 512, grace.GRACE_BF16),
])
def test_workspace_of_a_larger_batch_does_for_a_smaller_one(E, k, I, f, dt):
    """A serving loop sizes one buffer for its largest batch."""
    sizes = [grace.grace_workspace_bytes(T, E, k, I, 2048, f, 0, dt) for T in range(0, 1100)]
    assert all(a <= b for a, b in zip(sizes, sizes[1:]))
    # rows by slots are held for the batches that are laid out so: 32 tokens with more than 64 experts, 96, or 256 with k <= 2; 1024 choices
    el, most = 4 if dt == grace.GRACE_F32 else 2, min(32 if E > 64 else 96 if k > 2 else 256, 1024 // k) if max(E, I) <= 256 else 0
    assert sizes[most] >= min(32 << 20, most * min(E, I) * f * el)
    assert sizes[1099] <= max(min(32 << 20, most * min(E, I) * f * el), 1099 * k * f * el, 1 << 20) + 512


def test_caller_tensors_are_checked_before_a_kernel_writes_them():
    """Tensors that kernels of these calls write or read whole: too small or of another type is an error, not an access out of
    bounds.  (Tensors of the right size get as far as the check that they are on the device.)"""
    T, k, R, N, I, d, f = 6, 3, 4, 2, 5, 16, 8
    table = types.SimpleNamespace(R=R, N=N, I=I, E=I, handle=None)
    sizes = dict(rank_send_ptr=R + 1, rank_send_tok=T * k, node_send_ptr=N + 1, node_send_tok=T * k, expand=T * k)
    good = {n: torch.zeros(c, dtype=torch.int32) for n, c in sizes.items()}
    good["traffic"] = torch.zeros(4, dtype=torch.int64)
    ti = torch.zeros((T, k), dtype=torch.int32)
    with pytest.raises(ValueError, match="live on the GPU"):
        grace.grace_send_lists_fresh(table, 0, ti, tuple(good.values()))
    for name, t in good.items():
        for bad in (t[:-1], t.double()) + (() if name == "traffic" else (t.long(), None)):
            with pytest.raises(ValueError, match=name):
                grace.grace_send_lists_fresh(table, 0, ti, tuple({**good, name: bad}.values()))

    bf = torch.bfloat16
    a = dict(x=torch.zeros(T, d, dtype=bf), perm_pos=torch.zeros(T * k, dtype=torch.int32), perm_src=torch.zeros(T * k, dtype=torch.int32),
             xp=torch.zeros(T * k, d, dtype=bf), inst_off=torch.zeros(I + 1, dtype=torch.int32), k=k, w_gate=torch.zeros(2, f, d, dtype=bf),
             w_up=torch.zeros(2, f, d, dtype=bf), state=torch.zeros(8, dtype=torch.int32), ws=torch.zeros(1 << 20, dtype=torch.uint8))
    with pytest.raises(ValueError, match="live on the GPU"):
        grace.grace_expert_ffn_up_share_scatter(table, 0, **a)
    for name, bad, said in (("perm_pos", a["perm_pos"][:-1], "perm_pos"), ("perm_src", a["perm_src"].long(), "perm_src"), ("inst_off", a["inst_off"][:I], "inst_off"),
                            ("xp", a["xp"][:-1], "xp"), ("xp", a["xp"].float(), "xp"), ("w_up", a["w_up"][:1], "w_up"), ("x", a["x"].float(), "one dtype"),
                            ("w_gate", a["w_gate"].float(), "one dtype"), ("state", a["state"][:7], "state"), ("ws", a["ws"][:64], "workspace")):
        with pytest.raises(ValueError, match=said):
            grace.grace_expert_ffn_up_share_scatter(table, 0, **{**a, name: bad})


def test_caller_tensors_of_the_joined_calls_are_checked():
    """The halves of a step that are one launch with other work: as the calls that they stand for, and the result too."""
    T, k, I, d, f, n, bf = 6, 3, 5, 16, 64, 2, torch.bfloat16
    table = types.SimpleNamespace(R=4, N=2, I=I, E=I, handle=None)
    i32, row = lambda n: torch.zeros(n, dtype=torch.int32), lambda *s: torch.zeros(s, dtype=bf)
    ws = torch.zeros(grace.grace_workspace_bytes(T, I, k, I, d, f), dtype=torch.uint8)
    ws_shared = torch.zeros(grace.grace_workspace_bytes(T, 1, 1, 1, d, f, n), dtype=torch.uint8)
    both = dict(inst_off=i32(I + 1), w_down=row(2, d, f), shared_down=row(n, d, f), y=row(T * k, d), y_shared=row(T, d), state=i32(8), ws=ws,
                ws_shared=ws_shared)
    bad = [(name, bad, name) for name, bads in dict(
        inst_off=(i32(I), torch.zeros(I + 1, dtype=torch.int64), None), y=(row(T * k - 1, d), row(T * k, d).float()), y_shared=(row(T - 1, d), None),
        state=(i32(7), None)).items() for bad in bads]
    bad += [("ws", ws[:-1], "workspace"), ("ws_shared", ws_shared[:-1], "workspace"), ("ws", None, "workspace"), ("ws_shared", None, "workspace"),
            ("shared_down", row(n, d, f + 8), "shared"), ("shared_down", row(n, d, f).float(), "shared")]
    calls = ((grace.grace_dispatch_ffn_down_share, {**both, "perm_pos": i32(T * k), "topk_weight": torch.zeros(T, k), "out": row(T, d)},
              [("perm_pos", i32(T * k - 1), "perm_pos"), ("topk_weight", torch.zeros(T, k).double(), "topk_weight"), ("out", row(T - 1, d), "out"),
               ("out", row(T, d).float(), "out")]),
             (grace.grace_expert_shared_ffn_down, {**both, "T": T, "k": k}, []))
    for call, args, more in calls:
        with pytest.raises(ValueError, match="live on the GPU"):
            call(table, 0, **args)
        for name, tensor, said in bad + more:
            with pytest.raises(ValueError, match=said):
                call(table, 0, **{**args, name: tensor})
    up = dict(k=k, x=row(T, d), w_gate=row(2, f, d), w_up=row(2, f, d), state=i32(8), ws=ws, ws_shared=ws_shared)
    for call, args in ((grace.grace_dispatch_ffn_up_share, {**up, "logits": torch.zeros(T, I), "shared": (row(n, f, d), row(n, f, d))}),
                       (grace.grace_expert_shared_ffn_up_scatter, {**up, "perm_pos": i32(T * k), "perm_src": i32(T * k), "xp": row(T * k, d),
                                                                   "inst_off": i32(I + 1), "shared_gate": row(n, f, d), "shared_up": row(n, f, d)})):
        for name, tensor, said in (("ws", ws[:-1], "workspace"), ("ws", None, "workspace"), ("ws_shared", None, "workspace"), ("state", i32(7), "state")):
            with pytest.raises(ValueError, match=said):
                call(table, 0, **{**args, name: tensor})


def test_native_calls_refuse_what_the_binding_refuses():
    """Checked before the library is reached: no device, and no table, is needed."""
    calls = binding._native()
    logits, inst = torch.zeros(3, 4), torch.zeros((3, 2), dtype=torch.int32)
    refused = [(calls.route, (0, 4, 0, logits, 2, 1, None, None, 0, 0)), (calls.route, (0, 4, 0, logits.double(), 2, 1, None, None, 0, 0)),
               (calls.route, (0, 4, 0, logits[0], 2, 1, None, None, 0, 0)), (calls.permute, (0, 4, 4, 2, 1, inst, None, 0)),
               (calls.permute, (0, 4, 4, 2, 1, inst, logits.double(), 0)), (calls.send_lists, (0, 4, 4, 2, 1, 0, inst, 0)),
               (calls.route_permute, (0, 4, 2, 1, 0, logits, 2, None, 1, None, None, 0, 0)),
               (calls.route_permute, (0, 4, 2, 1, 0, logits, 2, logits[0], 1, None, None, 0, 0))]
    for f, args in refused:
        with pytest.raises(ValueError):
            f(*args)
    with pytest.raises(TypeError):
        calls.route(0, 4, 0, None, 2, 1, None, None, 0, 0)
    with pytest.raises(TypeError):
        calls.permute(0)


def test_library_loads_without_the_native_calls(tmp_path):
    """A tree without the module of the calls that allocate, and no compiler: the library loads, and the calls take the way through Python."""
    root = os.path.dirname(os.path.dirname(os.path.abspath(grace.__file__)))
    shutil.copytree(os.path.join(root, "include"), tmp_path / "include")
    shutil.copytree(os.path.join(root, "paper_2509_25041_amd"), tmp_path / "paper_2509_25041_amd",
                    ignore=shutil.ignore_patterns("_torch_calls*", "_build", "__pycache__"))
    program = """
import types, warnings, torch
import paper_2509_25041_amd as grace
table = types.SimpleNamespace(handle=types.SimpleNamespace(value=None), E=4, I=4, R=2, N=1)
grace.binding._stream = lambda: 0
assert grace.grace_workspace_bytes(64, 4, 2, 4) > 0
with warnings.catch_warnings(record=True) as said:
    warnings.simplefilter("always")
    for call in (lambda: grace.grace_route(table, 0, torch.zeros(3, 4), 2), lambda: grace.grace_permute(table, torch.zeros((3, 2), dtype=torch.int32), None),
                 lambda: grace.grace_route_permute(table, 0, torch.zeros(3, 4), 2, None), lambda: grace.grace_send_lists(table, 0, torch.zeros((3, 2), dtype=torch.int32))):
        try:
            call()
        except ValueError as e:
            assert "live on the GPU" in str(e), e
        else:
            raise AssertionError("not refused")
assert len([w for w in said if "native" in str(w.message)]) == 1
"""
    run = subprocess.run([sys.executable, "-c", program], cwd=tmp_path, env={**os.environ, "PATH": str(tmp_path), "PYTHONPATH": str(tmp_path)},
                         capture_output=True, text=True)
    assert run.returncode == 0, run.stderr[-2000:]


def test_native_calls_belong_to_one_interpreter():
    """The module is named and stamped for the Python and the torch that it is compiled against."""
    from paper_2509_25041_amd import build
    binding._native()
    assert build.CALLS.endswith(sysconfig.get_config_var("EXT_SUFFIX")) and binding._calls.__file__ == build.CALLS
    assert not build.calls_are_stale()
    with open(build.CALLS_STAMP) as fh:
        assert fh.read().strip() == build.calls_digest() != build.source_digest()
