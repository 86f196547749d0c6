"""Host-only checks of the C ABI library: it loads, exports every declared
entry point, and rejects bad parameters before touching a device."""
import math
import os
import re

import pytest

from paper_2202_05012_amd import supa

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_functions():
    names = []
    for h in sorted(os.listdir(os.path.join(ROOT, "include"))):
        if h.endswith(".h"):
            text = open(os.path.join(ROOT, "include", h)).read()
            text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
            names += re.findall(r"\b(supa_[a-z0-9_]+)\s*\(", text)
    return sorted(set(names))


def test_library_exports_every_declared_symbol():
    lib = supa.load()
    names = declared_functions()
    assert "supa_simulate" in names and "supa_init_geometry" in names
    for name in names:
        assert hasattr(lib, name), f"{name} declared in include/ but not exported"
    assert lib.supa_abi_version() == 6


def base_geom(**kw):
    g = dict(n_planes=20, z_first=1.0, dz=1.0, e_cut=0.1, angle_mode="rayleigh", angle_a=0.1,
             frac_lo=0.0, frac_hi=1.0, frac_bits=21, img_nx=32, img_ny=32, img_x0=-5.0,
             img_x1=5.0, img_y0=-5.0, img_y1=5.0)
    g.update(kw)
    return g


def test_validation_accepts_workload_parameters():
    supa.validate_geometry(base_geom(), supa.OUT_HITS | supa.OUT_IMAGES | supa.OUT_TREE)


@pytest.mark.parametrize("bad", [
    dict(n_planes=0), dict(n_planes=64), dict(dz=0.0), dict(dz=-1.0), dict(z_first=0.0),
    dict(e_cut=-0.1), dict(e_cut=math.nan), dict(frac_lo=0.8, frac_hi=0.2),
    dict(frac_hi=1.5), dict(frac_bits=32), dict(angle_a=math.inf),
    dict(p_stop=[0.7] * 20, p_split=[0.5] * 20), dict(p_split=[-0.1] * 20),
    dict(layer_of_plane=[25] * 20), dict(layer_of_plane=[-2] * 20),
    dict(img_nx=0), dict(img_x1=-5.0), dict(img_nx=4096), dict(img_y0=math.nan),
])
def test_validation_rejects(bad):
    with pytest.raises(supa.SupaError) as e:
        supa.validate_geometry(base_geom(**bad), supa.OUT_HITS | supa.OUT_IMAGES)
    assert e.value.status == 1


def test_unknown_output_bits_rejected():
    with pytest.raises(supa.SupaError):
        supa.validate_geometry(base_geom(), 64)


def test_angle_mode_names():
    with pytest.raises(KeyError):
        supa.make_geometry(base_geom(angle_mode="gaussian"), 1)


def test_shape_entry_points_reject_bad_arguments_on_the_host():
    import ctypes as C
    from paper_2202_05012_amd import shapes
    L = shapes._lib()
    fake = C.c_void_p(4096)                       # never dereferenced: rejected first
    assert L.supa_shower_shapes(None, 10, 65, fake, fake, 1, 100, fake, fake, fake, fake, fake,
                                fake, fake, 2062) == 1
    assert L.supa_shower_shapes(None, 10, 20, fake, fake, 0, 100, fake, fake, fake, fake, fake,
                                fake, fake, 2062) == 1
    assert L.supa_shower_shapes(None, 10, 20, fake, fake, 1, -1, fake, fake, fake, fake, fake,
                                fake, fake, 2062) == 1
    assert L.supa_shower_shapes(None, 10, 20, fake, fake, 1, 100, C.c_void_p(4100), fake, fake,
                                fake, fake, fake, fake, 2062) == 1     # misaligned hit array
    assert "aligned" in L.supa_shapes_last_error().decode()
    assert L.supa_shapes_work_ints(10) == 2062 and L.supa_shapes_work_ints(-1) == -1
    assert L.supa_shower_shapes(None, 10, 20, fake, fake, 1, 100, fake, fake, fake, fake, fake,
                                fake, fake, 2061) == 1     # work too short for 10 showers
    assert "work" in L.supa_shapes_last_error().decode()
    assert L.supa_w1_workspace_bytes(0, 10, 5, 5) == 0
    need = L.supa_w1_workspace_bytes(7, 100, 1000, 2000)
    assert need > 7 * 100 * 8
    args = lambda **kw: [kw.get(k, d) for k, d in (
        ("s", None), ("cols", 7), ("ref", fake), ("nr", 1000), ("ldr", 7), ("smp", fake),
        ("ns", 2000), ("lds", 7), ("bins", 100), ("g", None), ("ng", 0), ("w1", fake),
        ("gm", None), ("ws", fake), ("wsb", need))]
    assert L.supa_w1_normalized(*args(bins=0)) == 1
    assert L.supa_w1_normalized(*args(bins=4097)) == 1
    assert L.supa_w1_normalized(*args(ldr=6)) == 1
    assert L.supa_w1_normalized(*args(wsb=need - 1)) == 1
    assert L.supa_w1_normalized(*args(g=fake, ng=0)) == 1


def test_grid_entry_points_reject_bad_arguments_on_the_host():
    import ctypes as C
    from paper_2202_05012_amd import grids as GR
    L = GR._lib()
    assert GR.cells([(96, 3, -5, 5, -5, 5), (12, 12, -5, 5, -5, 5), (6, 12, -5, 5, -5, 5)]) == 504
    assert GR.cells([(0, 3, -5, 5, -5, 5)]) == -1
    assert GR.cells([(3, 3, 5, -5, -5, 5)]) == -1
    fake = C.c_void_p(4096)
    big = GR._grids([(128, 128, 0.0, 1.0, 0.0, 1.0)])
    assert L.supa_bin_grids(None, 10, 1, C.cast(big, C.c_void_p), 21, fake, fake, 1, 100, fake, fake,
                            fake, fake, fake) == 1
    ok = GR._grids([(8, 8, 0.0, 1.0, 0.0, 1.0)])
    assert L.supa_bin_grids(None, 10, 1, C.cast(ok, C.c_void_p), 40, fake, fake, 1, 100, fake, fake,
                            fake, fake, fake) == 1
    assert L.supa_bin_grids(None, 10, 17, C.cast(ok, C.c_void_p), 21, fake, fake, 1, 100, fake, fake,
                            fake, fake, fake) == 1


@pytest.mark.parametrize("bad", [dict(n_regions=5, region_r=[0.1, 0.2, 0.3, 0.4]),
                                 dict(n_regions=3, region_r=[0.2, 0.1]),
                                 dict(n_regions=2, region_r=[0.0])])
def test_ring_parameters_rejected(bad):
    R = bad["n_regions"]
    g = dict(base_geom(), **bad, p_stop=[0.0] * 20 * R, p_split=[1.0] * 20 * R)
    with pytest.raises(supa.SupaError):
        supa.validate_geometry(g)
    ok = dict(base_geom(), n_regions=3, region_r=[0.1, 0.2], p_stop=[0.0] * 60, p_split=[1.0] * 60)
    supa.validate_geometry(ok)


def call_outputs(n, **kw):
    """Fake device addresses (never dereferenced) for every output of a call."""
    names = ("hit_offsets", "hit_x", "hit_y", "hit_e", "hit_layer", "hit_key", "images",
             "node_offsets", "node_parent", "node_gen", "node_vx", "node_vy", "node_vz", "node_e",
             "node_key", "ledger", "counts")
    o = {k: 4096 * (i + 1) for i, k in enumerate(names)}
    o.update(hit_capacity=1000, node_capacity=1000, shower_capacity=n)
    o.update(kw)
    return o


ALL_OUT = supa.OUT_HITS | supa.OUT_IMAGES | supa.OUT_TREE | supa.OUT_KEYS


def test_call_validation_accepts_a_well_formed_call():
    supa.validate_call(base_geom(), ALL_OUT, 100, call_outputs(100))
    supa.validate_call(base_geom(), ALL_OUT, 100, call_outputs(250))
    supa.validate_call(base_geom(), supa.OUT_HITS, 0, call_outputs(0, ledger=None, counts=None))


@pytest.mark.parametrize("n,bad", [
    (100, dict(shower_capacity=99)),        # per-shower rows past the caller's arrays
    (100, dict(shower_capacity=0)),
    (1, dict(shower_capacity=-1)),
    (100, dict(ledger=None)), (100, dict(counts=None)),
    (100, dict(hit_offsets=None)), (100, dict(hit_x=None)), (100, dict(hit_key=None)),
    (100, dict(images=None)), (100, dict(node_offsets=None)), (100, dict(node_vz=None)),
    (100, dict(node_key=None)), (100, dict(hit_capacity=-1)), (100, dict(node_capacity=-5)),
    (-1, {}), (2 ** 31, dict(shower_capacity=2 ** 31)),
])
def test_call_validation_rejects_on_the_host(n, bad):
    with pytest.raises(supa.SupaError) as e:
        supa.validate_call(base_geom(), ALL_OUT, n, call_outputs(max(n, 0), **bad))
    assert e.value.status == 1
    if "shower_capacity" in bad and 0 < n < 2 ** 31:
        assert "shower_capacity" in str(e.value)


def test_call_validation_checks_parameters_too():
    with pytest.raises(supa.SupaError) as e:
        supa.validate_call(base_geom(dz=0.0), ALL_OUT, 10, call_outputs(10))
    assert e.value.status == 1


def test_binding_refuses_wrong_dtypes_and_short_outputs():
    """The binding's own size and type check, run on host tensors (no GPU):
    each per-shower and per-record tensor must have the element type the
    library writes and hold the call's showers or the stated capacity."""
    import torch
    sim = object.__new__(supa.Simulator)
    sim.geom, sim.L, sim.device = base_geom(), 20, torch.device("cpu")
    n = 10

    def outputs():
        return {"ledger": torch.zeros((n, 4), dtype=torch.int64), "counts": torch.zeros((n, 6), dtype=torch.int32),
                "hit_offsets": torch.zeros(n, dtype=torch.int64),
                "hit_x": torch.zeros(50), "hit_y": torch.zeros(50), "hit_e": torch.zeros(50),
                "hit_layer": torch.zeros(50, dtype=torch.int32), "hit_capacity": 50,
                "images": torch.zeros((n, 20, 32, 32))}

    sim._check_output_sizes(outputs(), n)
    assert sim._shower_capacity(outputs()) == n
    for name, bad in (("ledger", torch.zeros((n, 4), dtype=torch.int32)),
                      ("counts", torch.zeros((n, 6), dtype=torch.int64)),
                      ("hit_offsets", torch.zeros(n, dtype=torch.int32)),
                      ("hit_x", torch.zeros(50, dtype=torch.float64)),
                      ("hit_layer", torch.zeros(50, dtype=torch.float32)),
                      ("images", torch.zeros((n, 20, 32, 32), dtype=torch.float64))):
        o = outputs()
        o[name] = bad
        with pytest.raises(ValueError, match=name):
            sim._check_output_sizes(o, n)
    o = outputs()
    o["images"] = torch.zeros((n - 1, 20, 32, 32))
    with pytest.raises(ValueError, match="images"):
        sim._check_output_sizes(o, n)
    assert sim._shower_capacity(o) == n - 1


def test_judge_entry_points_reject_bad_arguments_on_the_host():
    import ctypes as C
    from paper_2202_05012_amd import surrogate as S
    L = S._lib()
    fake = C.c_void_p(4096)                       # never dereferenced: rejected first
    assert L.supa_w1_equal_workspace_bytes(-1, 3) == -1
    assert L.supa_w1_equal_workspace_bytes(10, 5000) == -1
    need = L.supa_w1_equal_workspace_bytes(1000, 20)
    assert need >= 2 * 2 * 1000 * 20 * 4
    args = lambda **kw: [kw.get(k, d) for k, d in (
        ("s", None), ("n", 1000), ("cols", 20), ("a", fake), ("lda", 20), ("b", fake), ("ldb", 20),
        ("w1", fake), ("work", fake), ("wb", need))]
    assert L.supa_w1_equal(*args(n=0)) == 1
    assert L.supa_w1_equal(*args(cols=0)) == 1
    assert L.supa_w1_equal(*args(lda=19)) == 1
    assert L.supa_w1_equal(*args(wb=need - 1)) == 1
    assert "workspace" in L.supa_surrogate_last_error().decode()
    assert L.supa_w1_equal(*args(b=None)) == 1
    assert L.supa_sort_columns(None, 100, 3, fake, 2, fake, fake, 1 << 20) == 1       # ld < cols
    assert L.supa_sort_columns(None, 0, 3, fake, 3, fake, fake, 0) == 0              # empty: nothing to do
    assert L.supa_occupied_counts(None, 10, 0, 16, fake, 0.1, fake) == 1


def test_train_step_rejects_what_the_loss_rejects():
    import ctypes as C
    from paper_2202_05012_amd import surrogate as S
    L = S._lib()
    fake = C.c_void_p(4096)                       # never dereferenced: rejected first
    ptrs = (C.c_void_p * 8)(*[4096] * 8)
    need = L.supa_mlp_train_workspace_bytes(64, 32, 1, 40)
    assert need > 0
    step = lambda s_clamp, mse: L.supa_mlp_train_step(None, 64, 32, 1, 40, fake, 32, fake, fake, 1.0, s_clamp, mse, ptrs,
                                                      ptrs, ptrs, ptrs, 1e-3, 0.9, 0.999, 1e-8, 1, fake, fake, need)
    loss = lambda s_clamp, mse: L.supa_nll_grad(None, 64, 20, fake, fake, fake, 1.0, s_clamp, mse, fake, fake)
    for call in (loss, step):
        for s_clamp in (-1.0, -1e-30, float("inf"), float("nan")):
            assert call(s_clamp, 1) == 1
            assert "s_clamp" in L.supa_surrogate_last_error().decode()
        assert call(20.0, 2) == 1
        assert "mse_mean" in L.supa_surrogate_last_error().decode()
