"""Host-side checks of the C ABI that need no GPU: the library loads and
exports every function include/normpre.h declares, the defaults follow the
paper's optimizer table, and argument validation returns the documented
codes without touching a device."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "normpre.h")


@pytest.fixture(scope="module")
def N():
    from paper_2609_36692_amd import normpre
    if not os.path.exists(normpre.LIB_PATH):
        from paper_2609_36692_amd import _build
        _build.build_library()
    normpre.load_library()
    return normpre


def _declared_functions():
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(normpre_[a-z_0-9]+)\s*\(", text)))


def test_header_declares_entry_points():
    names = _declared_functions()
    for required in ("normpre_init", "normpre_step", "normpre_destroy", "normpre_last_error"):
        assert required in names


def test_library_exports_every_declared_symbol(N):
    lib = ctypes.CDLL(N.LIB_PATH)
    missing = [n for n in _declared_functions() if not hasattr(lib, n)]
    assert not missing, f"not exported: {missing}"


def test_hparams_layout_matches_header(N):
    # The struct as the C library sees it: defaults written by C, read by ctypes.
    hp = N.normpre_default_hparams()
    assert abs(hp.lr - 6e-4) < 1e-9
    assert abs(hp.momentum - 0.95) < 1e-7
    assert abs(hp.weight_decay - 0.1) < 1e-7
    assert abs(hp.target_rms - 0.2) < 1e-7
    assert hp.ns_iters == 5
    assert [round(c, 4) for c in hp.ns_coeffs] == [3.4445, -4.775, 2.0315]
    assert (hp.rank, hp.oversample, hp.power_iters) == (32, 8, 1)
    assert hp.seed == 1337 and hp.step == 0 and hp.flags == 0
    assert ctypes.sizeof(N.normpre_hparams) == 80


def test_version(N):
    assert "gfx950" in N.normpre_version()


@pytest.mark.parametrize("variant,shapes,over,code", [
    (0, [(768, 2304)], {}, 0),
    (1, [(768, 2304), (3072, 768)], {}, 0),
    (2, [(8, 8)], {}, 0),                            # Muon reference step
    (3, [(8, 8)], {}, 0),                            # normalize-only reference step
    (4, [(8, 8)], {}, -1),
    (-1, [(8, 8)], {}, -1),
    (2, [(8, 8)], {"ns_iters": 0}, -1),
    (2, [(8, 40000)], {}, 0),                        # Muon has no row-active pass
    (3, [(8, 40000)], {}, -2),
    (0, [(0, 8)], {}, -1),
    (0, [(8, -1)], {}, -1),
    (0, [(8, 8)], {"ns_iters": 0}, -1),
    (0, [(8, 8)], {"ns_iters": 65}, -1),
    (1, [(8, 8)], {"rank": 0}, -1),
    (1, [(8, 8)], {"oversample": -1}, -1),
    (1, [(8, 8)], {"power_iters": 9}, -1),
    (0, [(8, 8)], {"lr": float("nan")}, -1),
    (0, [(8, 8)], {"lr": -1.0}, -1),
    (0, [(8, 8)], {"weight_decay": float("inf")}, -1),
    (0, [(8, 8)], {"flags": 64}, 0),                 # finite check
    (1, [(8, 8)], {"flags": 64}, 0),
    (2, [(8, 8)], {"flags": 64}, -1),                # not for the Muon step
    (0, [(8, 8)], {"flags": 128}, -1),               # unknown flag
    (0, [(8, 8)], {"norm_eps": 0.0}, -1),
    (0, [(8, 8)], {"orientation": 4}, -1),
    (1, [(8, 8)], {"flags": 32}, 0),                 # interaction source X
    (0, [(8, 8)], {"flags": 32}, -1),                # source X is NormPre-L only
    (1, [(8, 8)], {"flags": 32, "orientation": 3}, -1),
    (0, [(8, 8)], {"orientation": 3}, 0),            # both axes
    (1, [(8, 40000)], {"orientation": 3, "step": 1}, -2),  # both axes: the row pass needs short rows
    (0, [(8, 8)], {"flags": 256}, -1),               # unknown flag
    (1, [(100, 1000)], {"flags": 16}, 0),            # exact NormPre-L, a = 100
    (1, [(400, 1000)], {"flags": 16}, 0),            # exact above 384 rows: dense eigensolver
    (1, [(400, 1000)], {"flags": 16, "step": 1}, 0),
    (1, [(9000, 16)], {"flags": 16}, -2),            # exact needs a <= 8192
    (1, [(1000, 1000)], {"flags": 16, "rank": 400}, -2),  # exact above 384 rows: rank <= 384
    (1, [(1000, 300)], {"flags": 16, "step": 1}, 0), # column-active: a = 300
    (0, [(8, 8)], {"flags": 16}, -1),                # exact flag is NormPre-L only
    (0, [(8, 8)], {"flags": 4}, 0),                  # no tangent
    (1, [(8, 8)], {"flags": 8}, 0),                  # strict tangent
    (0, [(8, 8)], {"flags": 12}, -1),                # both tangent modes
    (0, [(8, 40000)], {}, -2),                       # row-active row too long
    (0, [(8, 40000)], {"orientation": 2}, 0),        # column-active is fine
    (0, [(8, 40000)], {"step": 1}, 0),               # t odd -> column-active
    (1, [(1024, 1024)], {"rank": 400}, -2),          # sketch width above 384
    (1, [(100, 1024)], {"rank": 400}, 0),            # l = min(100, 408)
    (0, [(1 << 21, 4)], {"orientation": 2}, -2),
    (0, [], {}, 0),
])
def test_validate_codes(N, variant, shapes, over, code):
    hp = N.normpre_default_hparams(**over)
    got, msg = N.normpre_validate(variant, shapes, hp)
    assert got == code, msg
    if code:
        assert msg


def test_validate_null_arguments(N):
    lib = N.load_library()
    hp = N.normpre_default_hparams()
    assert lib.normpre_validate(0, 1, None, ctypes.byref(hp), None, 0) == N.NORMPRE_ERR_INVALID_ARG
    assert lib.normpre_validate(0, 0, None, None, None, 0) == N.NORMPRE_ERR_INVALID_ARG
    assert lib.normpre_validate(0, -1, None, ctypes.byref(hp), None, 0) == N.NORMPRE_ERR_INVALID_ARG


def test_entry_points_reject_null_context(N):
    lib = N.load_library()
    hp = N.normpre_default_hparams()
    assert lib.normpre_step(None, 0, 0, None, None, None, None, ctypes.byref(hp), None) == \
        N.NORMPRE_ERR_NOT_INITIALIZED
    assert "null" in N.normpre_last_error(None)
    assert lib.normpre_debug_fetch(None, 0, 0, None, 0, None) == N.NORMPRE_ERR_NOT_INITIALIZED
    assert lib.normpre_kernel_stats(None, 0, None, None, None, None, None, 0) == N.NORMPRE_ERR_NOT_INITIALIZED
    assert lib.normpre_init(None, 0) == N.NORMPRE_ERR_INVALID_ARG
    lib.normpre_destroy(None)   # no-op
    assert lib.normpre_sketch_omega(1, 0, 0, 10, 4, None, None) == N.NORMPRE_ERR_INVALID_ARG


def test_init_without_gpu_reports_hip_error(N):
    import torch
    if torch.cuda.is_available():
        pytest.skip("a GPU is present")
    ctx = ctypes.c_void_p()
    assert N.load_library().normpre_init(ctypes.byref(ctx), 0) == N.NORMPRE_ERR_HIP
    assert not ctx.value
    assert "device" in N.normpre_last_error(None)


def test_binding_fails_loudly_without_library(tmp_path):
    from paper_2609_36692_amd import normpre
    with pytest.raises(RuntimeError):
        # A fresh load from a path with no library must raise, never fall back.
        saved = normpre._lib
        normpre._lib = None
        try:
            normpre.load_library(str(tmp_path / "missing.so"))
        finally:
            normpre._lib = saved


def test_header_constants_match_binding(N):
    """Every NORMPRE_* integer constant of include/normpre.h has the same value
    in the Python binding."""
    import re
    hdr = open(os.path.join(ROOT, "include", "normpre.h")).read()
    consts = dict(re.findall(r"#define\s+(NORMPRE_[A-Z_0-9]+)\s+\(?(-?\d+)u?\)?", hdr))
    assert consts, "no constants parsed"
    missing = [k for k in consts if not hasattr(N, k)]
    assert not missing, missing
    for k, v in consts.items():
        assert getattr(N, k) == int(v), (k, getattr(N, k), v)


def test_energy_split_host_matches_oracle(N):
    # Host-only entry point: no GPU involved.
    import numpy as np
    from oracle import normpre_oracle as O
    rng = np.random.default_rng(5)
    lam = np.sort(np.concatenate([rng.uniform(1.0, 30.0, 40), rng.uniform(0.0, 1.0, 60), [1.0, 0.0, -1e-9]]))[::-1]
    for count, r in [(len(lam), 32), (len(lam), 0), (50, 100), (0, 5)]:
        got = N.normpre_energy_split(lam, count, r)
        want = O.energy_split(lam, count, r)
        np.testing.assert_allclose(got, [want["top"], want["remain"], want["sub"], want["global"]], rtol=1e-13,
                                   atol=1e-13)
    with pytest.raises(N.NormPreError):
        N.normpre_energy_split(lam, -1, 3)


def test_sketch_workspace_holds_what_is_used_and_every_part_of_a_list(N):
    def need(shapes, rank):
        return N.normpre_workspace_size(N.NORMPRE_VARIANT_L, shapes, N.normpre_default_hparams(rank=rank))
    # Per matrix of 768 x 1024, l = 72 (both sides and l padded, 1024 and 128): Psi;
    # Omega, V (two fp16, two fp32 copies), Q and F; the split sums (at most 16);
    # l_pad^2 entries of 4 fp64 Gram slots, 2 fp64 of the Cholesky and 2 fp32
    # small matrices; statistics.  With 16 Gram slots it was 15.0 MB.
    lp, side = 128, 1024
    psi = 2 * 768 * side
    most = psi + lp * side * (2 + 2 * 2 + 2 * 4 + 2 + 2 + 16 * 4) + lp * lp * (4 * 8 + 2 * 8 + 2 * 4) + (1 << 18)
    assert need([(768, 1024)] * 96, 64) <= 96 * most
    # The number of slots falls as matrices are added (4 from 16 on here), the
    # workspace does not.
    for rank in (8, 32, 64, 80, 120):
        sizes = [need([(768, 6000)] * k, rank) for k in range(1, 40)]
        assert sizes == sorted(sizes)


def test_workspace_size_is_host_only_and_covers_both_orientations(N):
    hp = N.normpre_default_hparams()
    shapes = [(768, 2304), (3072, 768), (768, 768)]
    g = N.normpre_workspace_size(N.NORMPRE_VARIANT_G, shapes, hp)
    lv = N.normpre_workspace_size(N.NORMPRE_VARIANT_L, shapes, hp)
    assert g > 0 and lv > 0
    # the requirement covers t and t + 1, so it does not depend on t's parity
    hp.step = 1
    assert N.normpre_workspace_size(N.NORMPRE_VARIANT_G, shapes, hp) == g
    # more matrices never need less
    assert N.normpre_workspace_size(N.NORMPRE_VARIANT_G, shapes * 2, hp) >= g
    assert N.normpre_workspace_size(N.NORMPRE_VARIANT_G, [], hp) == 0
    with pytest.raises(N.NormPreError) as ei:
        N.normpre_workspace_size(N.NORMPRE_VARIANT_G, [(0, 5)], hp)
    assert ei.value.code == N.NORMPRE_ERR_INVALID_ARG
