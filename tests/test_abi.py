"""The C ABI without a GPU: the library loads, exports every symbol the header declares, and its
host-side helpers and argument validation behave as documented (validation happens before any
launch, so these calls never touch a device)."""
import ctypes
import os
import re

import pytest

import oracle
from _util import align256, attn_layout

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "pasa.h")


@pytest.fixture(scope="module")
def P():
    import paper_2604_12219_amd as P
    if not os.path.exists(P.lib_path()):
        from paper_2604_12219_amd.build import build
        build()
    P.load_library()
    return P


def declared_symbols():
    text = open(HEADER).read()
    return sorted(set(re.findall(r"PASA_API\s+[\w\s\*]+?\b(pasa_\w+)\s*\(", text)))


def test_every_declared_symbol_is_exported(P):
    names = declared_symbols()
    assert {"pasa_block_score", "pasa_route", "pasa_route_gumbel", "pasa_sparse_attn_fwd", "pasa_attn_dense_ref", "pasa_kv_stats",
            "pasa_sparse_attn_fwd_prepared", "pasa_topk_count", "pasa_strerror"} <= set(names)
    lib = ctypes.CDLL(P.lib_path())
    for n in names:
        assert hasattr(lib, n), f"{n} is declared in pasa.h but not exported"
    from paper_2604_12219_amd.pasa import EXPORTS
    assert set(EXPORTS) == set(names)
    # ... and nothing else is: the dynamic symbol table holds exactly the declared entry points
    import subprocess
    out = subprocess.run(["nm", "-D", "--defined-only", P.lib_path()], capture_output=True, text=True, check=True).stdout
    exported = {l.split()[-1] for l in out.splitlines() if " T " in l and l.split()[-1].startswith("pasa_")}
    assert exported == set(names), exported ^ set(names)


def test_product_has_no_cpu_fallback_and_does_not_import_the_oracle():
    src = ""
    pkg = os.path.join(ROOT, "paper_2604_12219_amd")
    for f in os.listdir(pkg):
        if f.endswith(".py"):
            src += open(os.path.join(pkg, f)).read()
    assert "import oracle" not in src and "from oracle" not in src
    assert "There is no CPU fallback" in src


def test_topk_count_matches_the_oracle_rule_and_rejects_bad_ratios(P):
    for nb in (1, 7, 16, 512, 1182, 1154):
        for keep in (1e-6, 0.05, 0.15, 0.2, 0.25, 0.5, 0.999, 1.0):
            assert P.topk_count(nb, keep) == oracle.topk_count(nb, keep)
    for bad in (0.0, -0.1, 1.0001, float("nan")):
        with pytest.raises(P.PasaError):
            P.topk_count(100, bad)
    with pytest.raises(P.PasaError):
        P.topk_count(0, 0.5)


def _shape(P, **kw):
    base = dict(B=1, H=2, n=8192, d=128, block=64, group=32, stride_n=128)
    base.update(kw)
    base.setdefault("stride_h", max(base["n"], 1) * base["stride_n"])
    base.setdefault("stride_b", base["H"] * base["stride_h"])
    return P.Shape(**base)


def test_shape_helpers_and_workspace_sizes(P):
    s = _shape(P)
    assert P.num_blocks(s) == 128 and P.mask_words(16) == 1 and P.mask_words(1182) == 37
    assert P.num_blocks(_shape(P, n=1000)) == 16  # ragged tail
    assert P.score_workspace_bytes(s) >= 2 * 2 * 128 * 128 * 4
    assert P.attn_workspace_bytes(_shape(P, group=4096)) > 0  # at least N_B blocks per group: one global matrix
    assert P.attn_workspace_bytes(s) > 0
    assert P.attn_workspace_bytes(_shape(P, group=0)) > 0
    # invalid shapes report 0 bytes
    assert P.attn_workspace_bytes(_shape(P, d=96)) == 0
    assert P.attn_workspace_bytes(_shape(P, group=48)) == 0
    assert P.attn_workspace_bytes(_shape(P, kv_slices=3)) == 0
    assert P.score_workspace_bytes(_shape(P, block=32)) == 0


def test_argument_validation_returns_before_any_launch(P):
    L = P.load_library()
    good = _shape(P).c()
    fake = ctypes.c_void_p(0x1000)  # 16-byte aligned, never dereferenced: every call below fails validation first
    big = ctypes.c_size_t(1 << 40)
    EINVAL, EUNSUPPORTED, EWORKSPACE, EALIGN = -1, -2, -3, -4

    def score(shape, q=fake, k=fake, out=fake, ws=fake, nbytes=big):
        return L.pasa_block_score(q, k, ctypes.byref(shape), None, out, ws, nbytes, None)

    assert score(good, q=None) == EINVAL
    assert score(good, out=None) == EINVAL
    assert score(good, nbytes=ctypes.c_size_t(16)) == EWORKSPACE
    assert score(good, q=ctypes.c_void_p(0x1004)) == EALIGN
    assert score(_shape(P, d=96).c()) == EUNSUPPORTED
    assert score(_shape(P, block=256).c()) == EUNSUPPORTED
    assert score(_shape(P, n=0).c()) == EINVAL
    assert score(_shape(P, stride_n=100).c()) == EINVAL
    assert score(_shape(P, stride_n=132).c()) == EALIGN
    assert score(_shape(P, scale=-1.0).c()) == EINVAL

    def route(scores=fake, bh=2, nb=16, k=4, amp=0.1, idx=fake):
        return L.pasa_route(scores, bh, nb, k, 7, ctypes.c_float(amp), idx, None, None)


    assert route(scores=None) == EINVAL
    assert route(k=0) == EINVAL and route(k=17) == EINVAL
    assert route(amp=-1.0) == EINVAL and route(amp=float("inf")) == EINVAL
    assert route(nb=1 << 20, k=4) == EUNSUPPORTED
    assert L.pasa_route_gumbel(None, 2, 16, 4, 7, ctypes.c_float(0.5), fake, None, None) == EINVAL
    assert L.pasa_route_gumbel(fake, 2, 16, 0, 7, ctypes.c_float(0.5), fake, None, None) == EINVAL
    assert L.pasa_route_gumbel(fake, 2, 16, 4, 7, ctypes.c_float(-0.5), fake, None, None) == EINVAL
    assert L.pasa_route_gumbel(fake, 2, 1 << 20, 4, 7, ctypes.c_float(0.5), fake, None, None) == EUNSUPPORTED

    def sparse(shape, q=fake, idx=fake, mask=fake, k=4, out=ctypes.c_void_p(0x2000), ws=fake, nbytes=big):
        return L.pasa_sparse_attn_fwd(q, fake, fake, ctypes.byref(shape), idx, mask, k, out, None, ws, nbytes, None)

    assert sparse(good, idx=None, mask=None) == EINVAL  # one of the two may be missing, not both
    assert sparse(good, idx=ctypes.c_void_p(0x1002)) == EALIGN
    assert sparse(good, k=0) == EINVAL and sparse(good, k=129) == EINVAL
    assert sparse(good, out=fake) == EINVAL  # output aliases an input
    assert sparse(good, nbytes=ctypes.c_size_t(0)) == EWORKSPACE
    assert sparse(_shape(P, group=48).c()) == EUNSUPPORTED
    assert sparse(_shape(P, group=-1).c()) == EINVAL
    assert sparse(_shape(P, kv_slices=12).c()) == EUNSUPPORTED
    # size limits of the approximation pass: more than 65,535 groups (one block per group on a long sequence)
    assert sparse(_shape(P, n=70_000 * 64, group=1).c()) == EUNSUPPORTED
    assert P.attn_workspace_bytes(_shape(P, n=70_000 * 64, group=32)) > 0  # 70,000 blocks in groups of 32 are within the limits
    assert sparse(_shape(P, H=65_535, n=16_000_000).c()) == EUNSUPPORTED  # workgroup count beyond 32 bits

    def check(idx=fake, mask=fake, bh=2, nb=16, k=4, n_bad=fake):
        return L.pasa_check_selection(idx, mask, bh, nb, k, n_bad, None)

    assert check(idx=None, mask=None) == EINVAL and check(n_bad=None) == EINVAL
    assert check(k=0) == EINVAL and check(k=17) == EINVAL and check(bh=0) == EINVAL
    assert check(idx=ctypes.c_void_p(0x1002)) == EALIGN
    assert L.pasa_attn_dense_ref(fake, fake, fake, ctypes.byref(good), None, None, fake, big, None) == EINVAL
    assert L.pasa_kv_stats(None, fake, ctypes.byref(good), fake, big, None) == EINVAL
    # the entry point that allocates nothing: shapes beyond its static scratch are refused on the host
    ESCRATCH = -6

    def static(shape, q=fake, idx=fake, k=4, out=ctypes.c_void_p(0x2000)):
        return L.pasa_sparse_attn_fwd_static(q, fake, fake, ctypes.byref(shape), idx, fake, k, out, None, None)

    wan14b = _shape(P, H=40, n=75_600).c()
    assert P.attn_workspace_bytes(_shape(P, H=40, n=75_600)) > P.STATIC_SCRATCH_BYTES
    assert static(wan14b) == ESCRATCH
    assert P.attn_workspace_bytes(_shape(P, H=12, n=32_760)) <= P.STATIC_SCRATCH_BYTES  # the 480p shape fits
    assert static(good, q=None) == EINVAL and static(good, k=0) == EINVAL and static(good, k=129) == EINVAL
    assert static(_shape(P, group=48).c()) == EUNSUPPORTED and static(_shape(P, d=96).c()) == EUNSUPPORTED
    assert b"static" in L.pasa_strerror(ESCRATCH)
    # the whole forward in one call
    fwd_bytes = L.pasa_forward_workspace_bytes
    assert fwd_bytes(ctypes.byref(good), 0.15) > P.attn_workspace_bytes(_shape(P)) + P.score_workspace_bytes(_shape(P))
    assert fwd_bytes(ctypes.byref(good), 0.0) == 0 and fwd_bytes(ctypes.byref(good), 1.5) == 0
    assert fwd_bytes(ctypes.byref(_shape(P, d=96).c()), 0.15) == 0

    def forward(shape, keep=0.15, q=fake, out=ctypes.c_void_p(0x2000), ws=fake, nbytes=big):
        return L.pasa_forward(q, fake, fake, ctypes.byref(shape), ctypes.c_double(keep), 7, ctypes.c_float(0.1), out, None, ws, nbytes, None)

    assert forward(good, keep=0.0) == EINVAL and forward(good, keep=float("nan")) == EINVAL
    assert forward(good, q=None) == EINVAL and forward(good, ws=None) == EINVAL
    assert forward(good, nbytes=ctypes.c_size_t(1024)) == EWORKSPACE
    assert forward(_shape(P, group=48).c()) == EUNSUPPORTED
    assert forward(_shape(P, n=5000 * 64).c()) == EUNSUPPORTED  # more key blocks than the routing kernel takes
    for code in (0, -1, -2, -3, -4, -5, -6, -99):
        assert isinstance(L.pasa_strerror(code), bytes) and len(L.pasa_strerror(code)) > 0


def test_whole_forward_checks_every_stage_before_the_first_launch(P):
    """an argument that only a later stage looks at is reported before anything is enqueued: without a device a launch would give PASA_EHIP.
    (CPU only: the pointers are no buffers)"""
    import torch
    if torch.cuda.is_available():
        pytest.skip("a launch that came too early would write through these pointers")
    L = P.load_library()
    EINVAL, EUNSUPPORTED, EWORKSPACE, EALIGN, EHIP = -1, -2, -3, -4, -5
    ok, big = dict(q=0x1000, k=0x1000, v=0x1000, out=0x2000), 1 << 40

    def buffers(shape, amp=0.1, k_sel=4, scores=0x3000, idx=0x4000, mask=0x5000, sws=0x6000, aws=0x7000, score_bytes=big, attn_bytes=big, **ptr):
        a = dict(ok, **ptr)
        return L.pasa_forward_buffers(a["q"], a["k"], a["v"], ctypes.byref(shape.c()), k_sel, 7, amp, scores, idx, mask, sws, score_bytes, aws, attn_bytes,
                                      a["out"], None, None)

    def single(shape, amp=0.1, **ptr):
        a = dict(ok, **ptr)
        return L.pasa_forward(a["q"], a["k"], a["v"], ctypes.byref(shape.c()), 0.15, 7, amp, a["out"], None, 0x6000, big, None)

    for shape in (_shape(P), _shape(P, group=0), _shape(P, H=40, n=75_600), _shape(P, d=64, n=1000), _shape(P, block=128, group=16)):
        nb = P.num_blocks(shape)
        for call in (buffers, single):
            assert call(shape) == EHIP  # (nothing to object to: the first launch)
            for name in ("q", "k", "v", "out"):
                assert call(shape, **{name: None}) == EINVAL, name
                assert call(shape, **{name: 0x1008}) == EALIGN, name
            assert call(shape, out=0x1000) == EINVAL  # output aliases an input
            for amp in (-1.0, float("inf"), float("nan")):
                assert call(shape, amp=amp) == EINVAL
        assert buffers(shape, k_sel=0) == EINVAL and buffers(shape, k_sel=-1) == EINVAL and buffers(shape, k_sel=nb + 1) == EINVAL
        assert buffers(shape, k_sel=nb) == EHIP
        for name in ("scores", "idx", "mask", "sws", "aws"):
            assert buffers(shape, **{name: None}) == EINVAL, name
        assert buffers(shape, scores=0x3004) == EALIGN and buffers(shape, sws=0x6004) == EALIGN and buffers(shape, aws=0x7004) == EALIGN
        assert buffers(shape, idx=0x4002) == EALIGN and buffers(shape, mask=0x5002) == EALIGN
        assert buffers(shape, score_bytes=P.score_workspace_bytes(shape) - 1) == EWORKSPACE
        assert buffers(shape, attn_bytes=attn_layout(shape)[0] - 1) == EWORKSPACE
        assert buffers(shape, score_bytes=P.score_workspace_bytes(shape), attn_bytes=attn_layout(shape)[0]) == EHIP
    for call in (buffers, single):
        assert call(_shape(P, group=48)) == EUNSUPPORTED and call(_shape(P, d=96)) == EUNSUPPORTED and call(_shape(P, n=5000 * 64)) == EUNSUPPORTED
        assert call(_shape(P, kv_slices=12)) == EUNSUPPORTED and call(_shape(P, scale=-1.0)) == EINVAL and call(_shape(P, n=0)) == EINVAL


def test_forms_of_the_attention_kernel(P):
    """pasa_attn_variant: what it refuses, the names of the binding in the order of the header, one shape of every form"""
    text = open(HEADER).read()
    names = dict((n.lower(), int(v)) for n, v in re.findall(r"PASA_ATTN_([A-Z_]+) = (\d+)", text))
    from paper_2604_12219_amd.pasa import ATTN_VARIANTS
    assert {n: i for i, n in enumerate(ATTN_VARIANTS)} == names
    for shape, k_sel, status in ((_shape(P), -1, -1), (_shape(P), 129, -1), (_shape(P, d=96), 0, -2), (_shape(P, group=48), 4, -2), (_shape(P, kv_slices=12), 4, -2)):
        assert P.load_library().pasa_attn_variant(ctypes.byref(shape.c()), k_sel) == status
        with pytest.raises(P.PasaError):
            P.attn_variant(shape, k_sel)
    assert P.attn_variant(_shape(P, group=48)) == "teams"  # (the dense path has no groups)
    assert P.attn_variant(_shape(P, n=1400)) == "teams" and P.attn_variant(_shape(P, H=12, n=32_760)) == "wide"
    assert P.attn_variant(_shape(P, n=32_768, kv_slices=8), 40) == "sliced" and P.attn_variant(_shape(P, H=4, n=4140), 10) == "deep"
    # walks of few tiles: dense (the last two sizes in front of the line and behind it), alone and in a grid that teams are too many for; blocks of 128
    assert [P.attn_variant(_shape(P, H=1, n=n)) for n in (64, 512, 513, 704, 705)] == ["short", "short", "whole", "whole", "teams"]
    assert [P.attn_variant(_shape(P, H=300, n=n)) for n in (64, 512)] == ["short", "short"]
    assert [P.attn_variant(_shape(P, H=1, n=n, d=64)) for n in (64, 448, 449, 960, 961)] == ["short", "short", "short_teams", "short_teams", "teams"]
    assert [P.attn_variant(_shape(P, H=300, n=n, d=64)) for n in (64, 960)] == ["short", "short"]
    assert [P.attn_variant(_shape(P, block=128), k) for k in (1, 5, 6, 64)] == ["short", "short", "whole", "whole"]
    assert [P.attn_variant(_shape(P, block=128, d=64), k) for k in (1, 31, 32, 64)] == ["short", "short", "whole", "whole"]
    assert [P.attn_variant(_shape(P, H=h, n=2048, d=64)) for h in (32, 64, 96, 128)] == ["wide", "whole", "whole", "whole"]
    assert [P.attn_variant(_shape(P, H=h, n=9900, d=64)) for h in (6, 12, 18, 40)] == ["wide", "wide", "whole", "whole"]
    assert [P.attn_variant(_shape(P, H=h, n=2048)) for h in (32, 64, 96, 128)] == ["wide"] * 4
    for d in (64, 128):  # nearly every block selected: the ring of eight tiles has nothing to gain
        assert [P.attn_variant(_shape(P, H=6, n=4140, d=d), k) for k in (7, 8, 56, 57, 65)] == ["whole", "deep", "deep", "whole", "whole"]
    assert P.attn_variant(_shape(P, H=40, n=75_600), 177) == "quad" and P.attn_variant(_shape(P, H=12, n=32_760), 102) == "whole"
    for shape, k_sel in ((_shape(P, H=40, n=32_760), 245), (_shape(P, H=24, n=47_628), 168), (_shape(P, H=40, n=60_480), 189), (_shape(P, H=12, n=68_040), 177),
                         (_shape(P, H=10, n=75_600), 177), (_shape(P, H=5, n=118_800), 279), (_shape(P, H=20, n=75_600), 177), (_shape(P, H=40, n=75_600), 130)):
        assert P.attn_variant(shape, k_sel) == "whole", shape  # what four query blocks a workgroup lost on where rows select alike
    assert P.attn_variant(_shape(P, H=40, n=75_600, group=16), 177) == "whole" and P.attn_variant(_shape(P, H=40, n=147_600, block=128), 58) == "whole"


def _forward_bytes(P, s, keep):
    bh, nb = s.B * s.H, P.num_blocks(s)
    return (align256(bh * nb * nb * 4) + align256(bh * nb * P.topk_count(nb, keep) * 4) + align256(bh * nb * -(-nb // 32) * 4) +
            align256(P.score_workspace_bytes(s)) + attn_layout(s)[0])


def _workspace_shapes(P):
    import random
    rng = random.Random(5)
    shapes = [_shape(P, H=1, n=64000), _shape(P, H=1, n=65536), _shape(P, H=1, n=32768), _shape(P, H=12, n=32760), _shape(P, H=2, n=1024, d=64),
              _shape(P, H=4, n=4140, group=64), _shape(P, H=1, n=1400, group=1000), _shape(P, H=1, n=15000, kv_slices=0),
              _shape(P, H=1, n=16384, kv_slices=8), _shape(P, H=1, n=20480, group=16, kv_slices=8)]
    for _ in range(60):
        shapes.append(_shape(P, B=rng.choice([1, 1, 2]), H=rng.randint(1, 40), n=int(2 ** rng.uniform(6, 17)), d=rng.choice([64, 128]),
                             block=rng.choice([64, 128]), group=rng.choice([0, 1, 2, 8, 16, 32, 32, 64, 96, 5000])))
    return shapes


def test_workspaces_of_the_plain_size_are_accepted(P):
    """room beyond the plain size (sums of small units) is an offer: a workspace without it, sized once for other shapes or by an
    earlier call, is taken by every entry point, and what the size query gives is never less"""
    L = P.load_library()
    fake, odd, out = ctypes.c_void_p(0x1000), ctypes.c_void_p(0x1004), ctypes.c_void_p(0x2000)
    EINVAL, EWORKSPACE, EALIGN = -1, -3, -4
    for s in _workspace_shapes(P):
        c, need = s.c(), attn_layout(s)[0]
        assert P.attn_workspace_bytes(s) >= need, s
        for nbytes, expect in ((need, EINVAL), (need - 1, EWORKSPACE)):  # (a null pointer is reported after the size)
            assert L.pasa_kv_stats(None, fake, ctypes.byref(c), fake, nbytes, None) == expect, s
            assert L.pasa_key_prior(None, fake, ctypes.byref(c), 1e-6, fake, fake, nbytes, None) == expect, s
            assert L.pasa_sparse_attn_fwd(None, fake, fake, ctypes.byref(c), fake, fake, 1, out, None, fake, nbytes, None) == expect, s
            assert L.pasa_sparse_attn_fwd_prepared(None, fake, fake, ctypes.byref(c), fake, fake, 1, out, None, fake, nbytes, None) == expect, s
        plain = _forward_bytes(P, s, 0.15)
        assert L.pasa_forward_workspace_bytes(ctypes.byref(c), 0.15) >= plain
        for nbytes, expect in ((plain, EALIGN), (plain - 1, EWORKSPACE)):  # (a misaligned key pointer is reported after the size)
            assert L.pasa_forward(fake, odd, fake, ctypes.byref(c), 0.15, 1, 0.1, out, None, fake, nbytes, None) == expect, s


def test_a_workspace_for_the_longest_clip_does_for_shorter_ones(P):
    L = P.load_library()
    fake, odd, out = ctypes.c_void_p(0x1000), ctypes.c_void_p(0x1004), ctypes.c_void_p(0x2000)
    longer, shorter = _shape(P, H=1, n=32896), _shape(P, H=1, n=32768)
    size = L.pasa_forward_workspace_bytes(ctypes.byref(longer.c()), 0.15)
    assert L.pasa_forward(fake, odd, fake, ctypes.byref(shorter.c()), 0.15, 1, 0.1, out, None, fake, size, None) == -4  # past the size check
    longer, shorter = _shape(P, H=1, n=65536), _shape(P, H=1, n=64000)
    assert L.pasa_kv_stats(None, fake, ctypes.byref(shorter.c()), fake, P.attn_workspace_bytes(longer), None) == -1


def test_static_scratch_takes_every_shape_of_at_most_its_size(P):
    """room for small units never keeps a shape from the static scratch"""
    for s in _workspace_shapes(P):
        if s.kv_slices <= 1:
            assert (attn_layout(s)[0] <= P.STATIC_SCRATCH_BYTES) == (P.attn_workspace_bytes(s) <= P.STATIC_SCRATCH_BYTES), s


def test_binding_raises_a_clear_error_when_the_library_is_missing(P, monkeypatch):
    import paper_2604_12219_amd.pasa as mod
    monkeypatch.setattr(mod, "_lib", None)
    monkeypatch.setattr(mod, "_LIB_PATH", "/nonexistent/libpasa_hip.so")
    with pytest.raises(RuntimeError, match="no CPU fallback"):
        mod.load_library()


def test_generated_mfma_sequences_are_up_to_date():
    """pasa_mfma_pipes.hpp is written by gen_mfma_pipes.py; the committed header must be what the generator emits"""
    import importlib.util
    csrc = os.path.join(ROOT, "paper_2604_12219_amd", "csrc")
    spec = importlib.util.spec_from_file_location("gen_mfma_pipes", os.path.join(csrc, "gen_mfma_pipes.py"))
    gen = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(gen)
    with open(os.path.join(csrc, "pasa_mfma_pipes.hpp")) as f:
        assert f.read() == gen.gen()


def test_sweeps_module_imports_without_a_gpu():
    import paper_2604_12219_amd.sweeps as sweeps
    assert callable(sweeps.main) and callable(sweeps.sweep_groups) and callable(sweeps.selection_histogram)


def test_budget_schedule_host_function_matches_oracle_and_rejects_bad_input():
    """pasa_budget_schedule is host-only: checked here without a GPU (Eq.9-11)"""
    import numpy as np
    import paper_2604_12219_amd as P
    g = np.random.default_rng(5)
    for n_prompts, n_steps, rho, dense in ((10, 50, 0.15, 0.2), (1, 7, 0.5, 0.0), (3, 33, 0.9, 0.3), (2, 5, 0.2, 1.0)):
        l1 = g.uniform(0.1, 2.0, size=(n_prompts, n_steps))
        np.testing.assert_allclose(P.budget_schedule(l1, rho, dense), oracle.budget_schedule(l1, rho, dense), rtol=1e-13)
    for bad in (dict(l1=[[1.0, -1.0]], rho=0.5), dict(l1=[[0.0, 0.0]], rho=0.5, dense_fraction=0.0), dict(l1=[[1.0, 2.0]], rho=0.0),
                dict(l1=[[1.0, float("nan")]], rho=0.5, dense_fraction=0.0), dict(l1=[[1.0, 2.0]], rho=0.5, dense_fraction=1.5)):
        with pytest.raises(P.PasaError):
            P.budget_schedule(**bad)
    # the schedule drives pasa_topk_count step by step
    r = P.budget_schedule(g.uniform(0.5, 1.5, size=(10, 50)), 0.15)
    ks = [P.topk_count(1182, x) for x in r]
    assert ks[:10] == [1182] * 10 and all(1 <= k <= 1182 for k in ks) and abs(sum(ks[10:]) - 0.15 * 1182 * 40) < 40


def test_binding_checks_that_the_strides_stay_inside_the_tensors():
    """host-side bounds check of the binding: a shape whose strides reach beyond a tensor's storage is refused before
    any library call (CPU tensors will do: the check never touches the data)"""
    import torch
    import paper_2604_12219_amd.pasa as mod
    q = torch.zeros((1, 2, 100, 64), dtype=torch.bfloat16)
    shape = mod.Shape.of(q)
    mod._check_extent(shape, q=q, k=q, v=None)  # fits exactly
    longer = mod.Shape(1, 2, 101, 64, 64, 32, shape.stride_b, shape.stride_h, shape.stride_n)
    with pytest.raises(ValueError, match="reach element"):
        mod._check_extent(longer, q=q)
    view = q[:, :, 10:]  # a view that starts later in the same storage has less room
    with pytest.raises(ValueError, match="reach element"):
        mod._check_extent(shape, q=view)
    mod._check_extent(mod.Shape.of(view), q=view)
    with pytest.raises(ValueError, match="bf16"):
        mod._check_extent(shape, q=q.float())


def test_forward_refuses_keys_and_values_of_another_layout_than_the_queries(P):
    """the kernels read K and V with the strides of Q: another layout would be misread without an error"""
    import torch
    q, k, v = (torch.zeros((1, 2, 128, 64), dtype=torch.bfloat16) for _ in range(3))
    other = torch.zeros((1, 128, 2, 64), dtype=torch.bfloat16).permute(0, 2, 1, 3)
    with pytest.raises(ValueError, match="k: strides"):
        P.forward(q, other, v, 0.5, 1, 0.1)
    with pytest.raises(ValueError, match="v: strides"):
        P.forward(q, k, other, 0.5, 1, 0.1)
    from paper_2604_12219_amd.pasa import _check_strides
    one = torch.zeros((1, 1, 128, 64), dtype=torch.bfloat16)  # a batch of one head: only the token stride counts
    _check_strides(P.Shape.of(one), k=one.as_strided((1, 1, 128, 64), (7, 9, 64, 1)))


def test_stream_handle_without_the_raw_getter(monkeypatch):
    """a torch without the raw-handle getter: the handle of torch.cuda.current_stream()"""
    import types

    import torch
    import paper_2604_12219_amd.pasa as binding
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=77))
    monkeypatch.setattr(binding, "_raw_stream", None)
    assert binding._stream() == 77


def test_header_is_plain_c(tmp_path):
    """include/pasa.h compiles as C99 with no HIP header in sight, and a C program links against the library by name"""
    import subprocess
    src = tmp_path / "use_pasa.c"
    src.write_text('#include "pasa.h"\n#include <stdio.h>\n'
                   'int main(void) { pasa_shape_t s = {1, 2, 1000, 128, 64, 32, 256000, 128000, 128, 0.0f, 0};\n'
                   '  printf("%d %d %zu %s\\n", pasa_num_blocks(&s), pasa_topk_count(16, 0.25), pasa_attn_workspace_bytes(&s) > 0 ? (size_t)1 : (size_t)0,'
                   ' pasa_strerror(PASA_ESCRATCH));\n  return 0; }\n')
    inc = os.path.join(ROOT, "include")
    subprocess.run(["gcc", "-std=c99", "-Wall", "-Werror", "-pedantic", "-fsyntax-only", "-I", inc, str(src)], check=True)
    import paper_2604_12219_amd as P
    exe = tmp_path / "use_pasa"
    libdir = os.path.dirname(P.lib_path())
    subprocess.run(["gcc", "-std=c99", "-I", inc, str(src), "-o", str(exe), "-L", libdir, "-l:libpasa_hip.so", f"-Wl,-rpath,{libdir}"],
                   check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout.split(maxsplit=3)
    assert out[:3] == ["16", "4", "1"] and "static" in out[3]
