"""Workspaces with no room for the one-launch iteration or the fused training step: the calls take them
as before and run level by level or layer by layer, with the same results."""
import ctypes

import numpy as np
import pytest

import games

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["f32", "f64"])
def test_solver_without_room_for_the_records(precision):
    import torch

    from paper_2408_14778_amd import Solver
    from paper_2408_14778_amd import _native as N
    from paper_2408_14778_amd.solver import GameArgs, make_config
    g = games.leduc_like(4, 2, deal="sequential")
    lib = N.load()
    args = GameArgs(g)
    cfg = make_config("cfr+", precision=precision)
    direct = make_config("cfr+", precision=precision, graph=False)
    full, small = N.CfrPlanInfo(), N.CfrPlanInfo()
    N.check(lib.cfr_plan(ctypes.byref(args.struct), ctypes.byref(cfg), ctypes.byref(full)))
    N.check(lib.cfr_plan(ctypes.byref(args.struct), ctypes.byref(direct), ctypes.byref(small)))
    assert small.workspace_bytes < full.workspace_bytes
    ref = Solver(g, "cfr+", precision=precision)
    T, R, S = games.random_state(g, seed=2, nonnegative=True)
    real = np.float64 if precision == "f64" else np.float32
    ref.set_state(T, R.astype(real), S.astype(real))
    ref.iterate(2)
    want = ref.exploitability()["expl"]
    ws = torch.empty(int(small.workspace_bytes), dtype=torch.uint8, device="cuda")
    h = ctypes.c_void_p()
    st = torch.cuda.current_stream().cuda_stream
    N.check(lib.cfr_build(ctypes.byref(args.struct), ctypes.byref(cfg),
                          ctypes.c_void_p(ws.data_ptr()), ctypes.c_size_t(ws.numel()),
                          ctypes.c_void_p(st), ctypes.byref(h)))
    s = Solver.__new__(Solver)
    s.__dict__.update(ref.__dict__)
    s._h, s.workspace = h, ws
    s.set_state(T, R.astype(real), S.astype(real))
    s.iterate(2)
    got = s.exploitability()["expl"]
    assert abs(got - want) <= (1e-12 if precision == "f64" else 1e-6) * abs(want)
    s.close()
    ref.close()
    N.check(lib.cfr_plan(ctypes.byref(args.struct), ctypes.byref(cfg), ctypes.byref(full)))
    rc = lib.cfr_build(ctypes.byref(args.struct), ctypes.byref(cfg), ctypes.c_void_p(ws.data_ptr()),
                       ctypes.c_size_t(int(small.workspace_bytes) - 256), ctypes.c_void_p(st),
                       ctypes.byref(h))
    assert N.ERRORS[rc] == "CFR_ENOMEM"


@pytest.mark.parametrize("B", [1, 31, 63, 512])
def test_network_without_room_for_the_fused_step(B):
    import torch

    from paper_2408_14778_amd import _native as N
    from paper_2408_14778_amd.warmstart import WarmStartNet
    F, H, A = 96, 256, 4
    rng = np.random.default_rng(6)
    x = torch.from_numpy(rng.standard_normal((B, F)).astype(np.float32)).to("cuda").to(torch.bfloat16)
    t = torch.softmax(torch.from_numpy(rng.standard_normal((B, A)).astype(np.float32)).to("cuda"), 1)
    m = torch.ones((B, A), device="cuda")
    a = WarmStartNet(F, H, A, max_batch=B, seed=4)
    params = a.params()
    need = a.lib.cfr_mlp_workspace_bytes(F, H, A, B)
    ws = torch.empty(need - 2 * H * H, dtype=torch.uint8, device="cuda")
    h = ctypes.c_void_p()
    N.check(a.lib.cfr_mlp_create(F, H, A, B, ctypes.c_void_p(ws.data_ptr()),
                                 ctypes.c_size_t(ws.numel()),
                                 ctypes.c_void_p(torch.cuda.current_stream().cuda_stream),
                                 ctypes.byref(h)))
    b = WarmStartNet.__new__(WarmStartNet)
    b.__dict__.update(a.__dict__)
    b._h = h
    p = np.ascontiguousarray(params, dtype=np.float32)
    N.check(a.lib.cfr_mlp_set_params(h, p.ctypes.data_as(ctypes.POINTER(ctypes.c_float)), p.size))
    for _ in range(2):
        la, lb = a.train_step(x, t, m, 1e-3), b.train_step(x, t, m, 1e-3)
        # (the loss is added in another order: B terms)
        assert abs(la - lb) <= B * 2.0 ** -23 * abs(la)
    assert np.array_equal(a.params(), b.params())
    assert torch.equal(a.forward(x), b.forward(x))
    b.close()
    a.close()
