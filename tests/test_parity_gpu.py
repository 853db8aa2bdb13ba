"""GPU parity: the HIP path (through the C-ABI) against the CPU oracle on the
same seeded inputs.

Global parity compares every output of a whole decode (and encode) with the
oracle's sequential raster decode.  The "wide" grids (40 x 120 latents) put 40
latents on a wavefront, three 16-row tiles, at K = 3 and at M = 320.  At the
full workload sizes the oracle decodes the top grid rows (an exact
sub-decode: every tap lies in the latent's row or above); for the 4K workload
65 rows, so that all five row tiles of its widest steps are compared element
by element.  In addition the oracle's per-latent function is evaluated on the
GPU's own final reconstruction at sampled latents (teacher-forced), which also
catches any tap read before it was written.  The oracle references are
computed on host threads while the GPU tests run (oracle_refs).
Bars: 1e-4 absolute on floats; symbols bit-exact; scale indices identical
except scales within 1e-4 relative of a table level (counted).
"""
import sys

import numpy as np
import pytest

from paper_2607_19082_amd import inputs, wf

import oracle_refs
from gpu_helpers import (compare, gpu_plan, make_case, max_rows_per_step, oracle_model, sample_latents,
                         teacher_forced, to_np, top_rows_check)

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

WIDE = [
    # (workload, H, W): 40 latents per wavefront, three 16-row tiles per step
    ("cheng-gmm3-1080p-120x68-m192", 40, 120),
    ("minnen-hr-4k-240x135-m320", 40, 120),
]
TOP_ROWS = {"cheng-gmm3-1080p-120x68-m192": 20, "minnen-relaxed-b8-120x68-m192": 3,
            "minnen-hr-4k-240x135-m320": 65}

if torch.cuda.is_available():
    oracle_refs.prefetch([("minnen-hr-4k-240x135-m320", None, None, None, 65, False)]
                         + [(n, H, W, None, None, False) for n, H, W in WIDE]
                         + [(n, None, None, None, r, False) for n, r in TOP_ROWS.items()])


@pytest.fixture(scope="module", autouse=True)
def device():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    wf.lib()  # fails loudly when the library is missing
    torch.cuda.set_device(0)
    return torch.device("cuda", 0)


def log(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def run_decode(cfg, w, table, psi, sym, driver="stream", precision="fp32"):
    plan = gpu_plan(cfg, w, table, driver, precision)
    psi_d = torch.from_numpy(psi).cuda()
    sym_d = torch.from_numpy(sym).cuda()
    out = plan.decode(psi_d, sym_d)
    plan.sync()
    res = to_np(out)
    plan.close()
    return res


def run_encode(cfg, w, table, psi, y, driver="stream", precision="fp32"):
    plan = gpu_plan(cfg, w, table, driver, precision)
    out, s = plan.encode(torch.from_numpy(psi).cuda(), torch.from_numpy(y).cuda())
    plan.sync()
    res, s = to_np(out), s.cpu().numpy()
    plan.close()
    return res, s


SMALL = [
    # (workload, H, W, B): ragged grids, at most 16 latents per wavefront
    # (one row tile; the wide cases below span three)
    ("minnen-16x16-m192", 7, 9, 1),
    ("minnen-16x16-m192", 5, 3, 2),
    ("cheng-gmm3-1080p-120x68-m192", 6, 11, 1),
    ("minnen-relaxed-b8-120x68-m192", 5, 7, 3),
    ("minnen-hr-4k-240x135-m320", 4, 10, 1),
]


DRIVERS = ["stream", "graph", "persistent", "dataflow", "resident"]


@pytest.mark.parametrize("driver", DRIVERS)
@pytest.mark.parametrize("name,H,W,B", SMALL)
def test_small_decode_encode(name, H, W, B, driver):
    log(f"case {name} H={H} W={W} B={B} driver={driver}")
    cfg, w, table, psi, sym = make_case(name, H=H, W=W, B=B)
    model = oracle_model(cfg, w, table)
    ref = model.decode(psi, sym)
    got = run_decode(cfg, w, table, psi, sym, driver)
    log(compare(got, ref, table, cfg["K"]))
    u = inputs.make_noise(cfg["B"], cfg["H"], cfg["W"], cfg["M"])
    y = inputs.encoder_input(sym, u, ref["mean"])
    got_e, s = run_encode(cfg, w, table, psi, y, driver)
    assert np.array_equal(s, sym)
    log(compare(got_e, ref, table, cfg["K"]))


@pytest.mark.parametrize("driver", DRIVERS)
@pytest.mark.parametrize("name", ["minnen-16x16-m192", "minnen-kodak-48x32-m192"])
def test_full_decode_encode(name, driver):
    log(f"case {name} full size driver={driver}")
    cfg, w, table, psi, sym = make_case(name)
    model = oracle_model(cfg, w, table)
    ref = model.decode(psi, sym)
    got = run_decode(cfg, w, table, psi, sym, driver)
    log(compare(got, ref, table, cfg["K"]))
    u = inputs.make_noise(cfg["B"], cfg["H"], cfg["W"], cfg["M"])
    y = inputs.encoder_input(sym, u, ref["mean"])
    got_e, s = run_encode(cfg, w, table, psi, y, driver)
    assert np.array_equal(s, sym)
    log(compare(got_e, ref, table, cfg["K"]))


@pytest.mark.parametrize("name,H,W,B", [
    ("cheng-gmm3-1080p-120x68-m192", 14, 24, 1),
    ("minnen-relaxed-b8-120x68-m192", 9, 16, 8),
    ("minnen-hr-4k-240x135-m320", 9, 20, 1),
])
@pytest.mark.parametrize("driver", ["graph", "persistent", "dataflow", "resident"])
def test_reduced_global(name, H, W, B, driver):
    log(f"case {name} reduced H={H} W={W} B={B} driver={driver}")
    cfg, w, table, psi, sym = make_case(name, H=H, W=W, B=B)
    ref = oracle_model(cfg, w, table).decode(psi, sym)
    got = run_decode(cfg, w, table, psi, sym, driver)
    log(compare(got, ref, table, cfg["K"]))


@pytest.mark.parametrize("name,H,W", WIDE)
@pytest.mark.parametrize("driver", ["graph", "persistent", "dataflow", "resident"])
def test_wide_global(name, H, W, driver):
    # every output of a decode whose wavefronts span three row tiles
    log(f"case {name} wide H={H} W={W} driver={driver}")
    cfg, w, table, psi, sym = make_case(name, H=H, W=W)
    assert max_rows_per_step(H, W, 3) == 40
    got = run_decode(cfg, w, table, psi, sym, driver)
    ref = oracle_refs.ref_decode(name, H, W).result()
    log(compare(got, ref, table, cfg["K"]))
    if driver == "graph":
        u = inputs.make_noise(cfg["B"], cfg["H"], cfg["W"], cfg["M"])
        y = inputs.encoder_input(sym, u, ref["mean"])
        got_e, s = run_encode(cfg, w, table, psi, y, driver)
        assert np.array_equal(s, sym)
        log(compare(got_e, ref, table, cfg["K"]))


@pytest.mark.parametrize("name,n", [
    ("cheng-gmm3-1080p-120x68-m192", 600),
    ("minnen-relaxed-b8-120x68-m192", 600),
    ("minnen-hr-4k-240x135-m320", 300),
])
@pytest.mark.parametrize("driver", ["graph", "persistent", "dataflow", "resident"])
def test_full_size_teacher_forced(name, n, driver):
    rows = TOP_ROWS[name]
    log(f"case {name} full size, top {rows} rows + teacher-forced sample of {n}, driver={driver}")
    cfg, w, table, psi, sym = make_case(name)
    got = run_decode(cfg, w, table, psi, sym, driver)
    ref = oracle_refs.ref_decode(name, rows=rows).result()
    log(top_rows_check(cfg, w, table, psi, sym, got, rows, ref=ref))
    model = oracle_model(cfg, w, table)
    lats = sample_latents(cfg, n)
    log(teacher_forced(cfg, got, psi, sym, model, lats, table))


def test_graph_replays_match_and_reuse_plan():
    # one graph plan, several calls with different buffers and both
    # directions, with eager work and syncs in between: every replay must
    # match the oracle
    cfg, w, table, psi, sym = make_case("minnen-16x16-m192", H=6, W=8, B=1)
    model = oracle_model(cfg, w, table)
    ref = model.decode(psi, sym)
    plan = gpu_plan(cfg, w, table, "graph")
    psi_d = torch.from_numpy(psi).cuda()
    sym_d = torch.from_numpy(sym).cuda()
    u = inputs.make_noise(cfg["B"], cfg["H"], cfg["W"], cfg["M"])
    y_d = torch.from_numpy(inputs.encoder_input(sym, u, ref["mean"])).cuda()
    for it in range(3):
        out = plan.decode(psi_d, sym_d)
        plan.sync()
        compare(to_np(out), ref, table, cfg["K"])
        junk = torch.randn(1000, device="cuda").sum().item()  # eager work between replays
        assert np.isfinite(junk)
        out_e, s = plan.encode(psi_d, y_d)
        plan.sync()
        assert np.array_equal(s.cpu().numpy(), sym)
        compare(to_np(out_e), ref, table, cfg["K"])
    plan.close()


@pytest.mark.parametrize("driver", ["graph", "persistent", "dataflow", "resident"])
def test_consecutive_calls_with_new_inputs(driver):
    # one plan, the same output buffers, two decodes of different symbols
    # (and an encode in between): nothing of an earlier call may be read back
    # as current data by a later one
    cfg, w, table, psi, sym = make_case("minnen-hr-4k-240x135-m320", H=9, W=20)
    sym2 = inputs.make_symbols(cfg["B"], cfg["H"], cfg["W"], cfg["M"], cfg["lap_b"], cfg["clip"], seed=7)
    model = oracle_model(cfg, w, table)
    refs = [model.decode(psi, s) for s in (sym, sym2)]
    plan = gpu_plan(cfg, w, table, driver)
    out = plan.alloc_out()
    psi_d = torch.from_numpy(psi).cuda()
    for rep in range(2):
        for s, ref in zip((sym, sym2), refs):
            plan.decode(psi_d, torch.from_numpy(s).cuda(), out=out)
            plan.sync()
            log(compare(to_np(out), ref, table, cfg["K"]))
        y = inputs.encoder_input(sym, inputs.make_noise(cfg["B"], cfg["H"], cfg["W"], cfg["M"]), refs[0]["mean"])
        _, s_out = plan.encode(psi_d, torch.from_numpy(y).cuda(), out=out)
        plan.sync()
        assert np.array_equal(s_out.cpu().numpy(), sym)
    plan.close()


@pytest.mark.parametrize("name,H,W", [
    ("minnen-16x16-m192", 15, 17),              # the hoisted product's 16-latent tiles
    ("minnen-kodak-48x32-m192", 33, 51),        # 32
    ("minnen-hr-4k-240x135-m320", 61, 101),     # 128
])
@pytest.mark.parametrize("value", [1e6, 1e12, np.inf, np.nan])
def test_resident_hoist_outlier(name, H, W, value):
    """An outlier or a value that is not finite in the last latent (no other
    depends on it) leaves every other latent's bits as they are, and reaches
    its own outputs as on the graph driver: per channel within 1e-4 of the
    sums of absolute products that the outlier's own channel makes (bounds
    from the weights' magnitudes)."""
    cfg, w, table, psi, sym = inputs.make_inputs(name, H=H, W=W)
    plain, psi = psi, psi.copy()
    psi[0, H - 1, W - 1, 3] = value
    got = {}
    for driver in ("graph", "resident"):
        plan = wf.Plan(w, table, H, W, 1, cfg["K"], driver=driver)
        sym_d = torch.from_numpy(sym).cuda()
        for what, p in (("plain", plain), ("outlier", psi)):
            out = plan.decode(torch.from_numpy(p).cuda(), sym_d)
            plan.sync()
            got[driver, what] = {k: v.cpu().numpy().reshape(H * W, -1) for k, v in out.items()}
        plan.close()
    for k in ("y_hat", "mean", "scale", "idx"):
        assert np.array_equal(got["resident", "plain"][k][:-1], got["resident", "outlier"][k][:-1]), k
    # |o| grows by at most |w3| |w2| |w1[:, 3]| |value| a channel (not finite:
    # what is left finite is a floor, the same on both)
    a = {k: np.abs(w[k].astype(np.float64)) for k in ("w1", "w2", "w3")}
    size = np.maximum(1.0, a["w3"] @ (a["w2"] @ a["w1"][:, 3]) * (abs(value) if np.isfinite(value) else 1.0))
    M = cfg["M"]
    for k, s in (("mean", size[:M]), ("scale", size[M:])):
        g, r = (got[d, "outlier"][k][-1].astype(np.float64) for d in ("graph", "resident"))
        assert np.array_equal(np.isfinite(g), np.isfinite(r)), k
        f = np.isfinite(g)
        assert (np.abs(g - r)[f] <= 1e-4 * s[f]).all(), k


@pytest.mark.parametrize("name,B,H,W", [
    ("minnen-16x16-m192", 1, 7, 9), ("minnen-16x16-m192", 2, 15, 17), ("minnen-kodak-48x32-m192", 1, 33, 51),
    ("minnen-hr-4k-240x135-m320", 1, 31, 47),
])
def test_resident_wide_range(name, B, H, W):
    """psi channels 1e-8 to 1e8 times the usual size, their layer-1 weights as
    much smaller or larger, and a channel of zeros with weights of 1e8: the
    products are the same as without the factors (powers of two), so every
    output keeps its bits -- nothing is scaled by what lies beside it."""
    cfg, w, table, psi, sym = inputs.make_inputs(name, H=H, W=W, B=B)
    psi[..., 5] = 0.0
    got = []
    for wide in (False, True):
        p, ww = psi.copy(), dict(w)
        if wide:
            ww["w1"] = w["w1"].copy()
            e = np.random.default_rng(13).integers(-27, 28, size=2 * cfg["M"])
            p *= np.ldexp(np.float32(1), e)
            ww["w1"][:, :2 * cfg["M"]] *= np.ldexp(np.float32(1), -e)
            ww["w1"][:, 5] = 1e8
        plan = wf.Plan(ww, table, H, W, B, cfg["K"], driver="resident")
        out = plan.decode(torch.from_numpy(p).cuda(), torch.from_numpy(sym).cuda())
        plan.sync()
        got.append({k: v.cpu().numpy() for k, v in out.items()})
        plan.close()
    for k in got[0]:
        assert np.array_equal(got[0][k], got[1][k]), k


def resident_grid(M, K, relaxed, nrep, parts, whole):
    """Workgroups of a resident fp32 plan with `parts` context parts (the last
    one included): per replica the column tiles of layers 1 and 2, two layer-3
    halves of each channel tile, the last context part and the other parts,
    four to a workgroup with `whole`."""
    tiles = lambda n: -(-n // 16)
    d1, d2, _ = inputs.widths(M, K)
    before = -(-(parts - 1) // 4) if whole else parts - 1
    return nrep * (tiles(d1) + tiles(d2) + 2 * tiles(M) + 2 * M // 64 * before + 2 * M // 32)


# tasks a step, and the workgroups that then hold each weight slice: from 3.5
# tasks four (bf16 from 4.5 three), below it, and at M = 320, two.  fp32 with M = 192
# keeps its 12 context parts (M = 128: 12), four to a workgroup where four
# replicas of them would not fit otherwise.
@pytest.mark.parametrize("name,B,H,W,precision,grid", [
    ("minnen-16x16-m192", 5, 15, 17, "fp32", (4, 12, True)),               # 5 tasks
    ("minnen-16x16-m192", 4, 16, 16, "fp32", (4, 12, True)),               # 4
    ("minnen-16x16-m192", 3, 16, 16, "fp32", (2, 12, False)),              # 3
    ("minnen-relaxed-b8-120x68-m192", 7, 17, 19, "fp32", (4, 12, True)),
    ("cheng-gmm3-1080p-120x68-m192", 3, 33, 40, "fp32", (4, 12, True)),
    ("minnen-16x16-m192", 6, 18, 17, "bf16", None),                        # three
    ("minnen-hr-4k-240x135-m320", 5, 15, 9, "fp32", (2, 8, False)),        # 5, two
])
def test_resident_replicas(name, B, H, W, precision, grid):
    """Plans with many tasks a step hold each weight slice in more workgroups,
    which take the tasks in turn; three calls through the same plan, each
    against the oracle."""
    cfg, w, table, psi, sym = make_case(name, H=H, W=W, B=B)
    log(f"resident replicas case {name} B={B} H={H} W={W} precision={precision}")
    ref = oracle_model(cfg, w, table, bf16=precision == "bf16").decode(psi, sym)
    plan = gpu_plan(cfg, w, table, driver="resident", precision=precision)
    slots = 2 * torch.cuda.get_device_properties(0).multi_processor_count
    if slots == 512:
        got = plan.trace(None)[1]
        if grid is not None:
            assert got == resident_grid(cfg["M"], cfg["K"], cfg["relaxed"], *grid)
        else:   # bf16: 3 x (40 + 32 + 24 column and channel tiles, 24 + 12 context slices); the rest hoists
            assert 3 * 132 <= got <= slots
    psi_d, sym_d = torch.from_numpy(psi).cuda(), torch.from_numpy(sym).cuda()
    for _ in range(3):
        out = plan.decode(psi_d, sym_d)
        plan.sync()
        compare(to_np(out), ref, table, cfg["K"], tol=1e-4 if precision == "fp32" else 1e-3)
    plan.close()


@pytest.mark.parametrize("name,B,H,W,precision,M", [
    ("minnen-16x16-m192", 5, 15, 17, "fp32", 192),                # four replicas, context parts of 8 and 9 k-blocks
    ("minnen-relaxed-b8-120x68-m192", 7, 17, 19, "fp32", 192),    # 6 and 7
    ("cheng-gmm3-1080p-120x68-m192", 3, 33, 40, "fp32", 192),
    ("minnen-16x16-m192", 6, 33, 20, "fp32", 128),                # four replicas, parts split over four waves
    ("minnen-16x16-m192", 6, 33, 20, "fp32", 64),
    ("minnen-16x16-m192", 6, 18, 17, "fp32", 160),                # three replicas
    ("minnen-hr-4k-240x135-m320", 5, 17, 9, "fp32", 320),
    ("minnen-16x16-m192", 6, 18, 17, "bf16", 192),
    ("minnen-16x16-m192", 6, 18, 17, "bf16", 256),                # three replicas leave no slots for the hoist in the launch
])
def test_resident_bits_alone_and_in_a_batch(name, B, H, W, precision, M):
    """An image's bits are the same in a batch, alone, beside other images and
    on a grid that goes on below it: a batch coded with the scale indices of
    one plan can be decoded image by image with another."""
    cfg = dict(inputs.workload(name), M=M)
    K, mask = cfg["K"], "relaxed" if cfg["relaxed"] else "full"
    w, table = inputs.make_weights(M, K), inputs.scale_table()
    psi = inputs.make_psi(B, H, W, M)
    psi[1] *= 1e4                                                  # (the others do not change with it)
    psi = torch.from_numpy(psi).cuda()
    sym = torch.from_numpy(inputs.make_symbols(B, H, W, M, cfg["lap_b"], cfg["clip"])).cuda()

    def call(p, s):
        plan = wf.Plan(w, table, p.shape[1], p.shape[2], p.shape[0], K, mask=mask, precision=precision, driver="resident")
        out = to_np(plan.decode(p.contiguous(), s.contiguous()))
        plan.sync()
        plan.close()
        return out

    batch = call(psi, sym)
    for b in (0, B - 1):
        one = call(psi[b:b + 1], sym[b:b + 1])
        for k in one:
            assert np.array_equal(one[k][0], batch[k][b]), (b, k)
    top = call(psi[:2, :H - 2], sym[:2, :H - 2])
    for k in top:
        assert np.array_equal(top[k], batch[k][:2, :H - 2]), k


def test_resident_batch_past_a_window():
    """A batch whose context parts together exceed one 2 GiB buffer window."""
    name, B = "minnen-relaxed-b8-120x68-m192", 11                  # 8033 tasks of 288 KiB
    cfg = inputs.workload(name)
    H, W, M = cfg["H"], cfg["W"], cfg["M"]
    w, table = inputs.make_weights(M, 1), inputs.scale_table()
    g = torch.Generator(device="cuda")
    g.manual_seed(21)
    psi = torch.randn((B, H, W, 2 * M), generator=g, device="cuda")
    sym = torch.round(2 * torch.randn((B, H, W, M), generator=g, device="cuda")).int()
    plan = wf.Plan(w, table, H, W, B, 1, mask="relaxed", driver="resident")
    out = plan.decode(psi, sym)
    plan.sync()
    plan.close()
    plan = wf.Plan(w, table, H, W, 1, 1, mask="relaxed", driver="resident")
    for b in (0, 7, B - 1):
        one = plan.decode(psi[b:b + 1].contiguous(), sym[b:b + 1].contiguous())
        plan.sync()
        for k in one:
            assert torch.equal(one[k][0], out[k][b]), (b, k)
    plan.close()
