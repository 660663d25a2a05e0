"""CPU checks of the C ABI: the library loads, exports every declared symbol,
validates its inputs and builds a consistent plan (no GPU needed)."""
import json
import os
import re

import numpy as np
import pytest

from paper_2104_10013_amd import ddpinn, workloads as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared():
    src = open(os.path.join(ROOT, "include", "ddpinn.h")).read()
    return sorted(set(re.findall(r"\b(ddp_[a-z_]+)\s*\(", src)))


def test_library_exports_every_declared_symbol():
    L = ddpinn.load_library()
    decl = _declared()
    assert len(decl) >= 18
    for name in decl:
        assert hasattr(L, name), name
    assert sorted(ddpinn.EXPORTED) == decl


def test_mfma_probe_rejects_bad_arguments():
    """Argument checks happen before any GPU call."""
    import ctypes as ct
    L = ddpinn.load_library()
    t = ct.c_double()
    assert L.ddp_mfma_probe(0, ct.byref(t)) == ddpinn.DDP_EINVAL
    assert L.ddp_mfma_probe((1 << 20) + 1, ct.byref(t)) == ddpinn.DDP_EINVAL
    assert L.ddp_mfma_probe(10, None) == ddpinn.DDP_EINVAL


def _plan(prob, tmp_path, **kw):
    pb = ddpinn.Problem(prob, plan_only=True, **kw)
    path = tmp_path / "plan.json"
    pb.plan_dump(path)
    d = json.load(open(path))
    pb.close()
    return d


def _item_cost(nets, q, kind, count):
    def c(n):
        return count * (1 + (nets[n]["depth"] - 1) * nets[n]["wclass"] ** 2 * 24 + 40 * nets[n]["wclass"])
    pair = nets[q]["pair"]
    return c(q) + (c(pair) * 4 / 3 if pair >= 0 and kind in (0, 2) else 0)


@pytest.mark.parametrize("name", ["c1_cpinn_poisson", "c2_xpinn_poisson", "c3_cpinn_burgers", "c4_xpinn_kovasznay",
                                  "c5_xpinn_inverse_diffusion", "burgers_st_xpinn_4x4", "burgers_st_cpinn_32x1",
                                  "burgers_st_hybrid_4x4", "ns_cpinn_kovasznay", "c5_table4_adaptive"])
def test_plan_covers_every_point_once(name, tmp_path):
    prob = W.make_problem(name, seed=0, scale=0.05 if name.startswith("c5") else 0.3)
    d = _plan(prob, tmp_path, chunk_points=100)
    nets = d["nets"]
    items = np.array(d["train_items"])
    q, kind, begin, count, iface, side, lrow, prow = (items[:, i] for i in range(8))
    assert (count > 0).all() and (count <= 128).all()   # chunk rounded up to the 64-point tile
    # residual, data and K-data points: each packed index in exactly one item
    for k, total in ((0, d["n_res"]), (1, d["n_dat"]), (3, d["n_aux"])):
        cover = np.zeros(total, int)
        for b, c in zip(begin[kind == k], count[kind == k]):
            cover[b:b + c] += 1
        assert (cover == 1).all()
    # activations; a problem with a general activation runs the kernels of
    # the class groups up to 80 and up to 112
    acts = {"tanh": 0, "sin": 1, "cos": 2}
    want_act = []
    for s in prob.subdomains:
        want_act += [(acts[s.act], int(s.adaptive))] * (1 if s.aux_widths is None else 2)
    assert [(n["act"], n["adaptive"]) for n in nets] == want_act
    assert [n["n_params"] for n in nets] == [W.param_count(wd, s.adaptive) for s in prob.subdomains
                                             for wd in ([s.widths] + ([s.aux_widths] if s.aux_widths else []))]
    if any(a != (0, 0) for a in want_act):
        assert all(l["wpmax"] in (80, 112) for l in d["launches"])
    # each interface keeps its own condition (the problem's unless set)
    want = [ddpinn._METHOD[e.method or prob.method] for e in prob.interfaces]
    assert [e["method"] for e in d["ifaces"]] == want
    # interface points: once per side
    cover = np.zeros((d["n_if"], 2), int)
    for b, c, s in zip(begin[kind == 2], count[kind == 2], side[kind == 2]):
        cover[b:b + c, s] += 1
    assert (cover == 1).all()
    # items of an interface side belong to that side's subdomain; K data to a K-network
    for row in items[kind == 2]:
        e = d["ifaces"][row[4]]
        assert nets[row[0]]["sd"] == (e["a"] if row[5] == 0 else e["b"])
    for row in items[kind == 3]:
        assert nets[row[0]]["pair"] == -1 and nets[row[0] - 1]["pair"] == row[0]
    # fused path: consecutive launches cover the items, descending cost within
    # each; an item is in the narrow launch iff every network it runs is <= 80
    cost = [_item_cost(nets, a, b, c) for a, b, c in zip(q, kind, count)]
    launches = d["launches"]
    assert launches[0]["begin"] == 0 and sum(l["count"] for l in launches) == len(items)
    for l in launches:
        seg = cost[l["begin"]:l["begin"] + l["count"]]
        assert all(seg[i] >= seg[i + 1] for i in range(len(seg) - 1))
    for l in launches[1:]:
        assert l["wpmax"] > 80 and launches[0]["wpmax"] <= 80
    # partial rows are disjoint, sized to the networks the item trains
    paired = np.array([nets[a]["pair"] >= 0 and b in (0, 2) for a, b in zip(q, kind)])
    size = np.array([nets[a]["gsize"] + (nets[nets[a]["pair"]]["gsize"] if pr else 0)
                     for a, pr in zip(q, paired)])
    order = np.argsort(prow)
    ends = prow[order] + size[order]
    assert (ends[:-1] <= prow[order][1:]).all() and ends[-1] == d["partial_floats"]
    # gradient rows: every item once under each network it trains, at that
    # network's part of the item's row
    ptr, ritem, rprow = d["net_row_ptr"], np.array(d["net_row_item"]), np.array(d["net_row_prow"])
    seen = []
    for n in range(len(nets)):
        for r in range(ptr[n], ptr[n + 1]):
            i = ritem[r]
            if q[i] == n:
                assert rprow[r] == prow[i]
            else:
                assert paired[i] and nets[q[i]]["pair"] == n and rprow[r] == prow[i] + nets[q[i]]["gsize"]
            seen.append((n, i))
    assert len(seen) == len(set(seen)) == len(items) + paired.sum()
    # loss rows: every item once under its subdomain
    lptr, lrows = d["sd_loss_ptr"], d["loss_rows"]
    assert sorted(lrows) == sorted(lrow.tolist())
    for sd in range(prob.n_sd):
        for r in lrows[lptr[sd]:lptr[sd + 1]]:
            assert nets[q[list(lrow).index(r)]]["sd"] == sd
    # parameter offsets follow the canonical layout sizes: [u | K] per subdomain
    sd_net = d["sd_net"]
    for sd, s in enumerate(prob.subdomains):
        u = nets[sd_net[sd]]
        assert u["n_params"] == W.param_count(s.widths, s.adaptive) and u["sd"] == sd
        assert u["wclass"] % 16 == 0 and u["wclass"] >= s.widths[1]
        if s.aux_widths is not None:
            k = nets[sd_net[sd] + 1]
            assert u["pair"] == sd_net[sd] + 1 and k["n_params"] == W.param_count(s.aux_widths, s.adaptive)
            assert k["poff"] == u["poff"] + u["n_params"]
        assert sd_net[sd + 1] - sd_net[sd] == (2 if s.aux_widths is not None else 1)


def _raw():
    L = ddpinn.load_library()
    import ctypes
    h = ctypes.c_void_p()
    coef = (ctypes.c_double * 1)(1.0)
    assert L.ddp_create(ctypes.byref(h), 1, 0, coef, 0) == 0
    return L, h, ctypes


def test_input_validation_codes():
    L, h, ct = _raw()
    lw = (ct.c_float * 4)(1, 1, 1, 1)
    sid = ct.c_int()
    good = (ct.c_int * 4)(2, 8, 8, 1)
    nl = (ct.c_int * 1)(4)
    assert L.ddp_add_subdomain(h, 1, nl, good, lw, 1e-3, ct.byref(sid)) == 0
    assert L.ddp_add_subdomain(h, 1, nl, good, lw, 1e-3, ct.byref(sid)) == 0
    bad = (ct.c_int * 4)(2, 8, 9, 1)   # uneven hidden widths
    assert L.ddp_add_subdomain(h, 1, nl, bad, lw, 1e-3, ct.byref(sid)) == ddpinn.DDP_EINVAL
    wide = (ct.c_int * 4)(2, 200, 200, 1)
    assert L.ddp_add_subdomain(h, 1, nl, wide, lw, 1e-3, ct.byref(sid)) == ddpinn.DDP_EINVAL
    two = (ct.c_int * 1)(4)
    assert L.ddp_add_subdomain(h, 2, two, good, lw, 1e-3, ct.byref(sid)) == ddpinn.DDP_EINVAL
    xy = np.array([[0.1, 0.2], [np.nan, 0.3]], np.float32)
    f = np.zeros(2, np.float32)
    rc = L.ddp_set_points(h, 0, 0, 2, xy.ctypes.data_as(ct.c_void_p), f.ctypes.data_as(ct.c_void_p), 0)
    assert rc == ddpinn.DDP_EINVAL and b"non-finite" in L.ddp_last_error()
    xy = np.array([[0.1, 0.2], [0.4, 0.3]], np.float32)
    nrm = (ct.c_float * 2)(1, 0)
    assert L.ddp_add_interface(h, 0, 5, 2, xy.ctypes.data_as(ct.c_void_p), nrm, 0, None) == ddpinn.DDP_EINVAL
    assert L.ddp_add_interface(h, 1, 1, 2, xy.ctypes.data_as(ct.c_void_p), nrm, 0, None) == ddpinn.DDP_EINVAL
    eid = ct.c_int(-1)
    assert L.ddp_add_interface(h, 0, 1, 2, xy.ctypes.data_as(ct.c_void_p), nrm, 0, ct.byref(eid)) == 0
    assert eid.value == 0
    assert L.ddp_set_interface_method(h, 1, ddpinn.DDP_CPINN) == ddpinn.DDP_EINVAL   # unknown interface
    assert L.ddp_set_interface_method(h, 0, 2) == ddpinn.DDP_EINVAL                  # unknown method
    assert L.ddp_set_interface_method(h, 0, ddpinn.DDP_CPINN) == 0
    # activation: validation, and D slopes per network once adaptive
    n = ct.c_int64()
    assert L.ddp_param_count(h, 1, ct.byref(n)) == 0 and n.value == W.param_count([2, 8, 8, 1])
    assert L.ddp_set_activation(h, 2, ddpinn.DDP_ACT_SIN, 1, 10.0) == ddpinn.DDP_EINVAL   # unknown subdomain
    assert L.ddp_set_activation(h, 1, 3, 1, 10.0) == ddpinn.DDP_EINVAL                    # unknown activation
    assert L.ddp_set_activation(h, 1, ddpinn.DDP_ACT_SIN, 2, 10.0) == ddpinn.DDP_EINVAL
    assert L.ddp_set_activation(h, 1, ddpinn.DDP_ACT_SIN, 1, 0.0) == ddpinn.DDP_EINVAL
    assert L.ddp_set_activation(h, 1, ddpinn.DDP_ACT_SIN, 1, float("nan")) == ddpinn.DDP_EINVAL
    assert L.ddp_set_activation(h, 1, ddpinn.DDP_ACT_COS, 1, 10.0) == 0
    assert L.ddp_param_count(h, 1, ct.byref(n)) == 0 and n.value == W.param_count([2, 8, 8, 1]) + 2
    assert L.ddp_set_activation(h, 1, ddpinn.DDP_ACT_SIN, 0, 10.0) == 0
    assert L.ddp_param_count(h, 1, ct.byref(n)) == 0 and n.value == W.param_count([2, 8, 8, 1])
    assert L.ddp_set_option(h, 99, 1) == ddpinn.DDP_EINVAL
    # calls that need a finalized problem
    ms4 = (ct.c_float * 4)()
    assert L.ddp_time_phases(h, 5, ms4) == ddpinn.DDP_ESTATE
    assert L.ddp_step(h, 1, None) == ddpinn.DDP_ESTATE
    assert L.ddp_sync(h) == ddpinn.DDP_ESTATE
    assert L.ddp_plan_dump(h, b"/tmp/x.json") == ddpinn.DDP_ESTATE
    assert L.ddp_plan(h) == 0
    assert L.ddp_destroy(h) == 0


def test_create_rejects_bad_combinations():
    L = ddpinn.load_library()
    import ctypes as ct
    h = ct.c_void_p()
    c = (ct.c_double * 1)(40.0)
    assert L.ddp_create(ct.byref(h), 0, 2, c, 1) == 0                   # cPINN + NS (Table 1 fluxes)
    assert L.ddp_destroy(h) == 0
    assert L.ddp_create(ct.byref(h), 1, 1, c, 0) == ddpinn.DDP_EINVAL   # Burgers without nu
    assert L.ddp_create(ct.byref(h), 3, 0, c, 0) == ddpinn.DDP_EINVAL
    neg = (ct.c_double * 1)(-1.0)
    assert L.ddp_create(ct.byref(h), 1, 2, neg, 1) == ddpinn.DDP_EINVAL
    assert L.ddp_create(ct.byref(h), 1, 2, c, 1) == 0
    assert L.ddp_destroy(h) == 0
    # inverse diffusion: XPINN only, two networks per subdomain, K data only there
    assert L.ddp_create(ct.byref(h), 0, 3, c, 0) == ddpinn.DDP_EINVAL
    assert L.ddp_create(ct.byref(h), 1, 3, c, 0) == 0
    lw = (ct.c_float * 4)(1, 1, 1, 1)
    one = (ct.c_int * 1)(4)
    w1 = (ct.c_int * 4)(2, 8, 8, 1)
    assert L.ddp_add_subdomain(h, 1, one, w1, lw, 1e-3, None) == ddpinn.DDP_EINVAL
    two = (ct.c_int * 2)(4, 3)
    w2 = (ct.c_int * 7)(2, 8, 8, 1, 2, 6, 2)     # K-network with two outputs
    assert L.ddp_add_subdomain(h, 2, two, w2, lw, 1e-3, None) == ddpinn.DDP_EINVAL
    w2 = (ct.c_int * 7)(2, 8, 8, 1, 2, 6, 1)
    assert L.ddp_add_subdomain(h, 2, two, w2, lw, 1e-3, None) == 0
    n = ct.c_int64()
    assert L.ddp_param_count(h, 0, ct.byref(n)) == 0 and n.value == W.param_count([2, 8, 8, 1]) + W.param_count([2, 6, 1])
    xy = np.array([[0.1, 0.2]], np.float32)
    v = np.ones(1, np.float32)
    assert L.ddp_set_points(h, 0, 2, 1, xy.ctypes.data_as(ct.c_void_p), v.ctypes.data_as(ct.c_void_p), 0) == 0
    assert L.ddp_add_subdomain(h, 2, two, w2, lw, 1e-3, None) == 0
    nrm = (ct.c_float * 2)(1, 0)
    assert L.ddp_add_interface(h, 0, 1, 1, xy.ctypes.data_as(ct.c_void_p), nrm, 0, None) == 0
    assert L.ddp_set_interface_method(h, 0, ddpinn.DDP_CPINN) == ddpinn.DDP_EINVAL   # no flux for the inverse problem
    assert L.ddp_set_interface_method(h, 0, ddpinn.DDP_XPINN) == 0
    assert L.ddp_destroy(h) == 0
    assert L.ddp_create(ct.byref(h), 1, 0, c, 0) == 0
    assert L.ddp_add_subdomain(h, 1, one, w1, lw, 1e-3, None) == 0
    assert L.ddp_set_points(h, 0, 2, 1, xy.ctypes.data_as(ct.c_void_p), v.ctypes.data_as(ct.c_void_p), 0) == ddpinn.DDP_EINVAL
    assert L.ddp_destroy(h) == 0


class _Recorder:
    """The library, with ddp_set_params recorded instead of called."""

    def __init__(self, lib):
        self.lib, self.calls = lib, []

    def __getattr__(self, name):
        return getattr(self.lib, name)

    def ddp_set_params(self, h, q, ptr, on_device):
        self.calls.append((q, ptr, on_device))
        return ddpinn.DDP_OK


def test_flat_parameters_of_the_host_take_the_host_path(monkeypatch):
    """A flat vector in host memory is handed over as host memory, subdomain by
    subdomain, and one that is too short reaches no call at all."""
    import torch
    pb = ddpinn.Problem(W.make_problem("c1_cpinn_poisson", seed=0, scale=0.1), plan_only=True)
    rec = _Recorder(ddpinn.load_library())
    monkeypatch.setattr(ddpinn, "_lib", rec)
    total = int(pb.offsets[-1])
    for n in (total, total + 5):
        rec.calls.clear()
        t = torch.arange(n, dtype=torch.float32)
        pb.set_params_flat(t)
        assert rec.calls == [(q, t.data_ptr() + 4 * int(pb.offsets[q]), 0) for q in range(pb.n_sd)]
    rec.calls.clear()
    for bad in (torch.zeros(0), torch.zeros(1), torch.zeros(total - 1), torch.zeros(1, total)):
        with pytest.raises(ddpinn.DDPError) as e:
            pb.set_params_flat(bad)
        assert e.value.code == ddpinn.DDP_EINVAL
    assert not rec.calls
    pb.close()
