"""The GEMM family's phased main loop (direct-to-LDS tiles, one barrier per
k-tile inside the products) against float64 products.

Every tile shape of its rule, and forms beyond it (k-tiles of 32, k-groups),
on sizes that leave partial tiles in every direction: rows, columns (multiples
of 8, as the path takes), contractions that 64 or 32 do not divide, fewer
k-tiles than stages, odd numbers of them, batches with a shared right operand.
The bound per element is the output's rounding plus the fp32 accumulation of K
products, K 2^-24 sum |a b| (each of the K additions rounds to 24 bits).
"""

import ctypes as C

import numpy as np
import pytest

torch = pytest.importorskip("torch")

SHAPES = ["256,256,2,4,1,64,2", "256,128,2,4,1,64,3", "128,128,2,2,1,64,2", "128,128,2,4,1,64,4", "128,96,2,2,1,64,2",
          "128,96,4,2,1,64,5", "128,64,4,2,1,64,5", "128,64,2,2,1,64,3", "64,128,2,2,1,64,3", "64,64,2,2,1,64,4",
          "32,64,2,2,1,64,6", "32,64,2,2,2,64,6", "256,256,2,4,1,32,5", "128,96,2,2,2,32,5"]
F32_SHAPES = ["64,128,2,2,1,32,2", "64,96,2,2,1,32,2", "64,64,2,2,1,32,2", "32,64,2,2,1,32,4", "32,32,2,2,1,32,4", "64,96,2,2,2,32,3",
              "32,64,2,2,2,32,6", "32,32,2,2,2,32,6", "128,128,2,4,1,32,4"]
# (the last number: the parts of the contraction that workgroups share)
SPLITS = ["32,64,2,2,2,64,6,2", "32,64,2,2,1,64,6,4", "64,64,2,2,1,64,4,3", "64,96,2,2,2,64,3,5", "128,128,2,4,1,64,4,8"]
F32_SPLITS = ["32,32,2,2,1,32,4,8", "32,32,2,2,2,32,6,3", "64,64,2,2,1,32,2,5", "32,64,2,2,2,32,6,4"]
# rows that end inside a 16-byte chunk among them
SIZES = [(300, 264, 200), (1, 8, 8), (257, 520, 64), (128, 96, 1000), (33, 72, 456), (130, 74, 322), (65, 2, 62), (40, 130, 2)]


def _graph(m, n, k, dtype, epi, batch=0, bt=False):
    from paper_2406_09465_amd._abi import Graph
    from paper_2406_09465_amd.graphs import Workload
    g = Graph()
    lead = (batch,) if batch else ()
    ids = {"A": g.input(dtype, lead + (m, k)), "W": g.input(dtype, ((batch,) if bt and batch else ()) + ((n, k) if bt else (k, n)))}
    names = ["A", "W"]
    if epi == "residual":
        ids["R"] = g.input(dtype, lead + (m, n))
        ids["b"] = g.input(dtype, (n,))
        names += ["R", "b"]
    if bt:  # the right operand is a transpose inside the kernel
        ids["Wb"] = g.op("transpose", [ids["W"]], dtype, perm=(0, 2, 1) if batch else (1, 0))
    elif batch:  # a right operand shared by the batch
        ids["Wb"] = g.op("reshape", [ids["W"]], dtype, shape=(1, k, n))
    ids["C"] = g.op("matmul", [ids["A"], ids["Wb" if batch or bt else "W"]], dtype)
    ids["out"] = ids["C"]
    prims = ([ids["Wb"]] if bt else []) + [ids["C"]]
    if epi == "residual":  # a value per column and one per element
        ids["Cb"] = g.op("add", [ids["C"], ids["b"]], dtype)
        ids["out"] = g.op("add", [ids["Cb"], ids["R"]], dtype)
        prims += [ids["Cb"], ids["out"]]
    g.output(ids["out"])
    g.finalize()
    return Workload("product", dtype, g, ids, names, ["out"]), [(prims, [ids["out"]])]


def _run(m, n, k, dtype, epi, batch=0, edit=None, seed=0, bt=False):
    from paper_2406_09465_amd.runner import TORCH_DTYPE, PlanRunner
    w, kernels = _graph(m, n, k, dtype, epi, batch, bt)
    r = PlanRunner(w, kernels=kernels)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    lead = (batch,) if batch else ()
    shapes = {"A": lead + (m, k), "W": (lead if bt else ()) + ((n, k) if bt else (k, n)), "R": lead + (m, n), "b": (n,)}
    x = {nm: torch.randn(shapes[nm], generator=gen, device="cuda").to(TORCH_DTYPE[dtype]) for nm in w.input_names}
    if edit:
        edit(x)
    r.ins = [x[nm] for nm in w.input_names]
    r.bind()
    r.launch_bound()
    torch.cuda.synchronize()
    x = {nm: v.double().cpu() for nm, v in x.items()}
    if bt:
        x["W"] = x["W"].transpose(-1, -2).contiguous()
    return r, x


def _check(r, x, k, dtype):
    out = r.outs[0].double().cpu()
    ref = x["A"] @ x["W"]
    mag = x["A"].abs() @ x["W"].abs()
    if "R" in x:
        ref = ref + x["b"] + x["R"]
        mag = mag + x["b"].abs() + x["R"].abs()
    eps = {"f16": 2.0 ** -11, "bf16": 2.0 ** -8, "f32": 2.0 ** -24}[dtype]
    bound = eps * ref.abs() * 1.01 + (k + 3) * 2.0 ** -24 * mag + 2.0 ** -24
    bad = (out - ref).abs() > bound
    assert not bool(bad.any()), f"{int(bad.sum())} of {bad.numel()} beyond the bound, worst {float(((out - ref).abs() / bound).max()):.2f}"


@pytest.mark.parametrize("cfg", SHAPES + F32_SHAPES + SPLITS + F32_SPLITS)
def test_phased_kernels_compile_without_spills(cfg, monkeypatch):
    """Each tile shape with a plain store and with a residual epilogue: no
    scratch, and M0 (the loads' LDS address, set in inline assembly the compiler
    does not see into) used by nothing else."""
    import os
    import subprocess
    import tempfile
    from paper_2406_09465_amd import codeobj
    from paper_2406_09465_amd._abi import Plan
    monkeypatch.setenv("KORCH_GEMM_PHASED", cfg)
    bm, bn, wm, wn, kg, bk, st, ks = (list(map(int, cfg.split(","))) + [1])[:8]
    f32 = cfg in F32_SHAPES + F32_SPLITS
    for epi in ("", "residual"):
        w, kernels = _graph(700, 520, 1032, "f32" if f32 else "bf16", epi)
        p = Plan(w.graph, kernels)
        p.compile()
        (grid, block, lds) = p.kernel_launch(0)
        assert grid[0] == -(-700 // bm) * -(-520 // bn) * ks and block[0] == 64 * wm * wn * kg and lds <= 160 * 1024
        assert "offen lds" in p.kernel_source(0)
        (res,) = codeobj.kernel_resources(p.kernel_code(0)).values()
        assert res["scratch"] == 0 and res["vgpr"] + res["agpr"] <= 512 // (block[0] // 256)
        objdump = "/opt/rocm/llvm/bin/llvm-objdump"
        if not os.path.exists(objdump):
            continue
        with tempfile.NamedTemporaryFile(suffix=".co") as f:
            f.write(p.kernel_code(0))
            f.flush()
            dis = subprocess.run([objdump, "-d", "--mcpu=gfx950", f.name], capture_output=True, text=True, check=True).stdout
        ins = [ln.split("//")[0].split() for ln in dis.splitlines() if ln.startswith("\t")]
        m0 = [i for i, w in enumerate(ins) if "m0" in [t.strip(",") for t in w]]
        assert m0 and all(ins[i][:2] == ["s_mov_b32", "m0,"] and ins[i + 1][0] == "s_nop" and ins[i + 2][-1] == "lds" for i in m0)


def test_phased_epilogue_that_spills_takes_smaller_tiles():
    """Three operands of the output's shape spill beside the accumulators of 256 x
    256 tiles; the kernel is generated again with 256 x 128."""
    from paper_2406_09465_amd import codeobj
    from paper_2406_09465_amd._abi import Graph, Plan
    g = Graph()
    a, b = g.input("bf16", (16384, 1024)), g.input("bf16", (1024, 4096))
    rest = [g.input("bf16", (16384, 4096)) for _ in range(3)] + [g.input("bf16", (4096,)) for _ in range(3)]
    prims = [g.op("matmul", [a, b], "bf16")]
    for i, r in enumerate(rest[3:] + rest[:3]):
        prims.append(g.op("add" if i < 3 else "mul", [prims[-1], r], "bf16"))
    g.output(prims[-1])
    g.finalize()
    p = Plan(g, [(prims, [prims[-1]])])
    p.compile()
    (res,) = codeobj.kernel_resources(p.kernel_code(0)).values()
    assert res["scratch"] == 0 and "offen lds" in p.kernel_source(0)
    assert p.kernel_launch(0)[0][0] == 16384 // 256 * 4096 // 128


# Plans whose tensors fill the static scratch of allocation-free execution, but
# not together with a split's partial sums: the hidden activation alone is 512 x
# 32000 fp16 = 32,768,000 of 33,488,896 bytes.
NEAR_LIMIT = dict(m=512, d=192, h=32000)


def test_workgroup_splits_keep_callers_workspace():
    """A long product of few tiles splits its contraction over workgroups, also
    where the plan with the split's partial sums is past the static scratch (the
    caller brings the workspace)."""
    from paper_2406_09465_amd import graphs
    static_ws = 33488896
    p = graphs.build("mlp", m=64, d=768, h=3072).plan("layered")
    assert "split_" in p.kernel_source(2) and p.workspace_bytes() <= static_ws
    for sizes in (NEAR_LIMIT, dict(m=512, d=192, h=40960)):
        p = graphs.build("mlp", **sizes).plan("layered")
        assert "split_" in p.kernel_source(2) and p.workspace_bytes() > static_ws


@pytest.mark.gpu
def test_workgroup_splits_keep_plans_allocation_free():
    """Allocation-free execution of a plan that fits the static scratch only
    without splits runs it without them; one that does not fit either way is
    refused."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2406_09465_amd import graphs
    from paper_2406_09465_amd._abi import KorchError, pointer_array
    from paper_2406_09465_amd.runner import PlanRunner
    from synthetic import workloads as W
    for sizes in (NEAR_LIMIT, dict(m=512, d=192, h=40960)):
        print(f"\n[case] near the static scratch {sizes}", flush=True)
        r = PlanRunner(graphs.build("mlp", **sizes), "layered")
        r.set_inputs(W.inputs("mlp", **sizes))
        r.launch()
        torch.cuda.synchronize()
        ref = r.outs[0].double()
        out = torch.zeros_like(r.outs[0])
        args = (pointer_array([t.data_ptr() for t in r.ins]), pointer_array([out.data_ptr()]), torch.cuda.current_stream().cuda_stream)
        if sizes is not NEAR_LIMIT:
            with pytest.raises(KorchError) as e:
                r.plan.execute_noalloc(*args)
            assert e.value.code == -22
            continue
        for _ in range(3):
            out.zero_()
            r.plan.execute_noalloc(*args)
            torch.cuda.synchronize()
            # the same products in another order of fp32 sums, rounded to fp16 once
            err = (out.double() - ref).abs()
            assert float((err - 2.0 ** -10 * ref.abs()).max()) <= 2.0 ** -10 * float(ref.abs().mean())


@pytest.mark.parametrize("switch,product", [("KORCH_GEMM_SCHED=0", (1024, 1024, 1024)), ("KORCH_GEMM_FULL_CTILE=1", (1024, 1024, 1024)),
                                            ("KORCH_LDS_BANK_SHIFT=0", (1024, 1024, 1024)), ("KORCH_SPLITK_WGS=32", (64, 64, 8192))])
def test_switches_of_the_older_loops_take_them(switch, product, monkeypatch):
    """Ablation switches that only the older loops have act on products that run
    the phased loop without them."""
    from paper_2406_09465_amd._abi import Plan
    w, kernels = _graph(*product, "f16", "")
    assert "offen lds" in Plan(w.graph, kernels).kernel_source(0)
    monkeypatch.setenv(*switch.split("="))
    p = Plan(w.graph, kernels)
    assert "offen lds" not in p.kernel_source(0)
    if "WGS" in switch:
        (grid, _, _) = p.kernel_launch(0)
        assert grid[0] * grid[1] * grid[2] <= 32


@pytest.mark.parametrize("switch", [
    "KORCH_GEMM_PHASED=128,128,0,2,1,64,2", "KORCH_GEMM_PHASED=128,128,2,2,1,0,2", "KORCH_GEMM_PHASED=0,128,2,2,1,64,2",
    "KORCH_GEMM_PHASED=128,-128,2,2,1,64,2", "KORCH_GEMM_PHASED=128,128,2,2,0,64,2", "KORCH_GEMM_PHASED=128,128,-2,-2,1,64,2",
    "KORCH_GEMM_PHASED=128,128,2,2,1,64,1000000000", "KORCH_GEMM_PHASED=1073741824,128,2,2,1,64,2",
    "KORCH_GEMM_CFG=0,128,32,2,2", "KORCH_GEMM_CFG=128,0,32,2,2", "KORCH_GEMM_CFG=128,128,32,-2,-2", "KORCH_GEMM_CFG=-128,128,32,2,2",
    "KORCH_GEMM_CFG=128,128,0,2,2"])
def test_inconsistent_tile_switches_are_ignored(switch):
    """In a process of its own (the first forms ended it with a division by zero)."""
    import os
    import subprocess
    import sys
    code = """
from paper_2406_09465_amd._abi import Graph, Plan
g = Graph()
a, b = g.input("f16", (700, 1032)), g.input("f16", (1032, 520))
c = g.op("matmul", [a, b], "f16")
g.output(c)
g.finalize()
p = Plan(g, [([c], [c])])
grid, block, lds = p.kernel_launch(0)
assert min(grid + block) > 0 and block[0] in (256, 512) and lds <= 160 * 1024
"""
    var, val = switch.split("=")
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", code], env={**os.environ, var: val}, cwd=root, capture_output=True, text=True)
    assert r.returncode == 0, (r.returncode, r.stderr[-300:])


def test_phased_selection():
    """Plain products take the path; rows that do not start on dwords and small
    short 16-bit products do not."""
    from paper_2406_09465_amd._abi import Plan

    def phased(m, n, k, dtype):
        w, kernels = _graph(m, n, k, dtype, "")
        p = Plan(w.graph, kernels)
        return "offen lds" in p.kernel_source(0)

    assert phased(4096, 1024, 1024, "bf16") and phased(1576, 384, 1536, "f16") and phased(301, 264, 1000, "f16")
    assert phased(2048, 768, 3072, "f32") and phased(49, 101, 37, "f32") and phased(512, 510, 1022, "bf16")
    assert not phased(4096, 1024, 1021, "f16") and not phased(4096, 1023, 1024, "f16") and not phased(512, 512, 128, "f16")


@pytest.mark.gpu
@pytest.mark.parametrize("size", SIZES, ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("cfg", SHAPES + SPLITS)
def test_phased_product(cfg, size, monkeypatch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    monkeypatch.setenv("KORCH_GEMM_PHASED", cfg)
    m, n, k = size
    for dtype, epi, batch, bt in (("f16", "", 0, False), ("bf16", "residual", 0, True), ("f16", "residual", 3, False)):
        print(f"\n[case] phased {cfg} {size} {dtype} {epi} batch {batch} bt {bt}", flush=True)
        r, x = _run(m, n, k, dtype, epi, batch, seed=m + n + k, bt=bt)
        assert "offen lds" in r.plan.kernel_source(0)
        _check(r, x, k, dtype)
        first = r.outs[0].clone()
        for _ in range(5):
            r.launch_bound()
        torch.cuda.synchronize()
        assert torch.equal(first.view(torch.int16), r.outs[0].view(torch.int16))


@pytest.mark.gpu
@pytest.mark.parametrize("size", [(300, 264, 200), (1, 4, 4), (129, 100, 36), (70, 96, 1000), (33, 68, 452), (65, 33, 97), (50, 1, 1),
                                  (34, 71, 191)],
                         ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("cfg", F32_SHAPES + F32_SPLITS)
def test_phased_f32_product(cfg, size, monkeypatch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    monkeypatch.setenv("KORCH_GEMM_PHASED", cfg)
    m, n, k = size
    for epi, batch, bt in (("", 0, True), ("residual", 3, False), ("", 2, True)):
        print(f"\n[case] phased f32 {cfg} {size} {epi} batch {batch} bt {bt}", flush=True)
        r, x = _run(m, n, k, "f32", epi, batch, seed=m + n + k, bt=bt)
        assert "offen lds" in r.plan.kernel_source(0)
        _check(r, x, k, "f32")
        first = r.outs[0].clone()
        for _ in range(5):
            r.launch_bound()
        torch.cuda.synchronize()
        assert torch.equal(first, r.outs[0])


@pytest.mark.gpu
@pytest.mark.parametrize("size", [(4096, 1024, 1024), (2048, 768, 3072), (1000, 1000, 1000), (64, 512, 4096), (5000, 96, 264)],
                         ids=lambda s: "x".join(map(str, s)))
def test_phased_default_choice(size):
    """The shapes the rule takes by itself (long contractions in two halves among them)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    m, n, k = size
    print(f"\n[case] phased default {size}", flush=True)
    r, x = _run(m, n, k, "f16", "residual", seed=5)
    assert "offen lds" in r.plan.kernel_source(0)
    _check(r, x, k, "f16")


# What the tile rule takes by itself at the edges of its terms: (m, n, k, dtype,
# epilogue, batch) and (tile rows, tile columns, k-tile, split over workgroups),
# or None where a product keeps the older loops.  One k-tile and three k-steps
# over more than a round of tiles, k-tiles of half a chunk row (16-bit and fp32)
# with a ragged end, many fp32 tiles in two stages, sixteen parts of a
# contraction, narrow outputs and one-step contractions.
CHOICES = [((2100, 520, 64, "f16", "residual", 0), (64, 64, 64, False)), ((2100, 520, 40, "bf16", "", 0), (64, 64, 64, False)),
           ((6900, 1000, 64, "f16", "", 0), (128, 128, 64, False)), ((4400, 1160, 64, "bf16", "", 0), (64, 128, 64, False)),
           ((2100, 520, 96, "f16", "residual", 0), (64, 64, 32, False)), ((700, 520, 90, "bf16", "", 5), (64, 64, 32, False)),
           ((2500, 2600, 160, "f16", "", 0), (128, 128, 32, False)), ((2500, 2600, 222, "bf16", "residual", 0), (128, 128, 32, False)),
           ((3100, 1100, 40, "f32", "", 0), (64, 64, 16, False)), ((3100, 1100, 71, "f32", "residual", 0), (64, 64, 16, False)),
           ((3100, 1100, 96, "f32", "residual", 0), (32, 64, 32, False)), ((70, 72, 20002, "f16", "", 0), (32, 64, 64, True)),
           ((21, 37, 9000, "f32", "residual", 0), (32, 32, 32, True)), ((16, 64, 1344, "bf16", "", 8), (32, 64, 64, True)),
           ((436, 2976, 5624, "bf16", "", 0), (128, 96, 64, True)), ((5000, 16, 104, "f16", "", 16), None),
           ((33000, 30, 66, "bf16", "", 0), None), ((3000, 1500, 32, "f16", "", 0), None), ((70000, 12, 40, "f32", "", 0), None)]


@pytest.mark.parametrize("product,tile", CHOICES, ids=lambda c: "x".join(map(str, c or ("older",))))
def test_phased_tile_rule(product, tile):
    import re
    from paper_2406_09465_amd import codeobj
    from paper_2406_09465_amd._abi import Plan
    w, kernels = _graph(*product)
    p = Plan(w.graph, kernels)
    p.compile()
    src = p.kernel_source(0)
    assert ("offen lds" in src) == (tile is not None)
    (res,) = codeobj.kernel_resources(p.kernel_code(0)).values()
    assert res["scratch"] == 0
    if tile:
        eb = 4 if product[3] == "f32" else 2
        got = [int(re.search(e, src)[1]) for e in (r"m0 = \(i64\)tm \* (\d+)", r"n0 = \(i64\)tn \* (\d+)", r"\(unsigned\)kt \* (\d+)")]
        assert (got[0], got[1], got[2] // eb, "split_ =" in src) == tile


# Products whose workgroups first touch the later part of the right operand: the
# MLP block's second product, ragged rows, columns and contraction, a transposed
# operand, the shortest contraction and the fewest rows; and one row less.
TOUCHES = [(4096, 768, 3072, "f16", False), (2600, 770, 2122, "bf16", False), (2997, 744, 2050, "f16", True), (2560, 832, 2048, "bf16", False)]


@pytest.mark.parametrize("product", TOUCHES, ids=lambda c: "x".join(map(str, c)))
def test_phased_touch_stays_inside_the_operand(product):
    """The touched dwords, over every workgroup and thread, lie in the right
    operand, and cover each of its cache lines from the first touched one on."""
    import re
    from paper_2406_09465_amd._abi import Plan
    m, n, k, dtype, bt = product
    w, kernels = _graph(m, n, k, dtype, "residual", bt=bt)
    p = Plan(w.graph, kernels)
    src, (grid, block, _) = p.kernel_source(0), p.kernel_launch(0)
    per, per2, lines, first, per3 = map(int, re.search(
        r"if \(tid < (\d+) && \(i64\)wg \* (\d+) \+ tid < (\d+)LL\) touch_ = \*\(const unsigned\*\)\(\(const char\*\)pB_ \+ (\d+)LL \+ "
        r"\(\(i64\)wg \* (\d+) \+ tid\) \* 128\);", src).groups())
    assert per == per2 == per3 <= block[0] and grid[0] * per >= lines
    assert first % 4 == 0 and first + (lines - 1) * 128 + 4 <= 2 * n * k <= first + lines * 128
    w, kernels = _graph(2559, n, k, dtype, "residual", bt=bt)
    assert "touch_" not in Plan(w.graph, kernels).kernel_source(0)


@pytest.mark.gpu
@pytest.mark.parametrize("product", TOUCHES, ids=lambda c: "x".join(map(str, c)))
def test_phased_touch_products(product):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    m, n, k, dtype, bt = product
    print(f"\n[case] phased touch {product}", flush=True)
    r, x = _run(m, n, k, dtype, "residual", seed=k, bt=bt)
    assert "touch_" in r.plan.kernel_source(0)
    full, r.outs = r.outs, [r.outs[0][::23]]
    _check(r, {nm: v[::23] if nm in ("A", "R") else v for nm, v in x.items()}, k, dtype)
    r.outs = full
    _repeat(r, f"touch {product}")


@pytest.mark.gpu
@pytest.mark.parametrize("product", [c for c, _ in CHOICES], ids=lambda c: "x".join(map(str, c)))
def test_phased_tile_rule_products(product):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    m, n, k, dtype, epi, batch = product
    print(f"\n[case] phased rule {product}", flush=True)
    r, x = _run(m, n, k, dtype, epi, batch, seed=m + k)
    first = r.outs[0].clone()
    for _ in range(5):
        r.launch_bound()
    torch.cuda.synchronize()
    assert torch.equal(first, r.outs[0])
    step = max(1, m // 200)  # rows enough to meet every kind of tile
    r.outs = [r.outs[0][..., ::step, :]]
    _check(r, {nm: v[..., ::step, :] if nm in ("A", "R") else v for nm, v in x.items()}, k, dtype)


@pytest.mark.gpu
def test_phased_nonfinite_rows_stay_apart():
    """A contraction that 64 does not divide: the chunks past a row's end are
    the next row's, and must not reach this row's sums even when they are
    infinite or NaN."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")

    def edit(x):
        x["A"][1::2] = float("inf")
        x["A"][3::4, 7] = float("nan")

    print("\n[case] phased nonfinite", flush=True)
    for k in (1000, 1002, 998):  # the last two end inside a chunk
        r, x = _run(130, 136, k, "f16", "", edit=edit)
        out = r.outs[0].double().cpu()
        ref = x["A"][0::2] @ x["W"]
        assert bool(torch.isfinite(out[0::2]).all()) and np.allclose(out[0::2], ref, rtol=2e-3, atol=0.15)
        assert not bool(torch.isfinite(out[1::2]).any())

    def edit_w(x):  # rows of the transposed operand
        x["W"][1::2] = float("nan")

    r, x = _run(70, 136, 37, "f32", "", edit=edit_w, bt=True)
    out = r.outs[0].double().cpu()
    assert np.allclose(out[:, 0::2], x["A"] @ x["W"][:, 0::2], rtol=1e-5, atol=1e-4) and bool(torch.isnan(out[:, 1::2]).all())


# Convolutions that the direct kernel does not take, as implicit GEMMs of the
# phased loop: k-tiles of 64 and of 32 channels, every filter size, images
# smaller than a tile, more workgroups than pixels, a per-channel epilogue.
CONVS = [("f16", 52, 52, 128, 256, 3), ("bf16", 9, 7, 256, 48, 5), ("f16", 33, 130, 96, 256, 3), ("f32", 31, 17, 64, 40, 3),
         ("bf16", 64, 64, 192, 96, 1), ("f32", 20, 20, 32, 256, 5), ("f16", 100, 100, 160, 128, 3)]
# Channels that end half a k-tile short on small maps, whose 32-row tiles have
# fewer blocks of half a k-tile than waves.
HALF_CONVS = [("f16", 14, 14, 96, 64, 3), ("f16", 20, 20, 160, 64, 3), ("bf16", 26, 26, 96, 128, 3), ("f16", 52, 52, 96, 128, 3),
              ("bf16", 57, 23, 96, 256, 3), ("f16", 40, 40, 96, 256, 5), ("f32", 40, 40, 48, 128, 3), ("f32", 13, 13, 80, 64, 3)]
CONVS += HALF_CONVS


@pytest.mark.parametrize("case", HALF_CONVS, ids=lambda c: "x".join(map(str, c)))
def test_phased_convolution_of_half_k_tiles(case):
    from paper_2406_09465_amd import graphs
    dtype, hh, ww, cin, cout, k = case
    assert "offen lds" in graphs.build("conv", dtype=dtype, hh=hh, ww=ww, cin=cin, cout=cout, k=k).plan("fused").kernel_source(0)


# Strides and paddings other than the workload's (1 and k / 2).
@pytest.mark.gpu
@pytest.mark.parametrize("case", [("f16", 30, 41, 64, 96, 3, 2, 1), ("bf16", 30, 41, 64, 96, 3, 2, 0), ("f16", 25, 25, 96, 64, 3, 1, 0),
                                  ("f32", 19, 33, 64, 40, 3, 2, 1), ("f16", 28, 27, 128, 72, 1, 2, 0), ("bf16", 23, 31, 96, 128, 5, 3, 2),
                                  ("f16", 11, 40, 64, 64, 3, 1, 3)], ids=lambda c: "x".join(map(str, c)))
def test_phased_convolution_strides(case):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2406_09465_amd._abi import Graph
    from paper_2406_09465_amd.graphs import Workload
    from paper_2406_09465_amd.runner import TORCH_DTYPE, PlanRunner
    dtype, hh, ww, cin, cout, k, stride, pad = case
    print(f"\n[case] phased conv strides {case}", flush=True)
    g = Graph()
    ids = {"X": g.input(dtype, (hh, ww, cin)), "W": g.input(dtype, (k, k, cin, cout)), "b": g.input(dtype, (cout,))}
    ids["C"] = g.op("conv2d", [ids["X"], ids["W"]], dtype, stride=stride, pad=pad)
    ids["out"] = g.op("add", [ids["C"], ids["b"]], dtype)
    g.output(ids["out"])
    g.finalize()
    r = PlanRunner(Workload("conv", dtype, g, ids, ["X", "W", "b"], ["out"]), kernels=[([ids["C"], ids["out"]], [ids["out"]])])
    assert "offen lds" in r.plan.kernel_source(0)
    gen = torch.Generator(device="cuda").manual_seed(hh + cin)
    r.ins = [torch.randn(s, generator=gen, device="cuda").to(TORCH_DTYPE[dtype]) for s in ((hh, ww, cin), (k, k, cin, cout), (cout,))]
    r.bind()
    r.launch_bound()
    torch.cuda.synchronize()
    x, w, b = (t.double().cpu() for t in r.ins)
    conv = lambda u, v: torch.nn.functional.conv2d(u.permute(2, 0, 1)[None], v.permute(3, 2, 0, 1), stride=stride, padding=pad)[0].permute(1, 2, 0)
    ref, mag = conv(x, w) + b, conv(x.abs(), w.abs()) + b.abs()
    eps = {"f16": 2.0 ** -11, "bf16": 2.0 ** -8, "f32": 2.0 ** -24}[dtype]
    bound = eps * ref.abs() * 1.01 + (k * k * cin + 1) * 2.0 ** -24 * mag + 2.0 ** -24
    err = (r.outs[0].double().cpu() - ref).abs()
    assert not bool((err > bound).any()), f"worst {float((err / bound).max()):.2f}"


@pytest.mark.gpu
@pytest.mark.parametrize("case", CONVS, ids=lambda c: "x".join(map(str, c)))
def test_phased_convolution(case):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from oracle import configs as OC
    from oracle.graph import run_unfused
    from paper_2406_09465_amd import graphs
    from paper_2406_09465_amd.runner import PlanRunner
    from tests.helpers import TOL, close, inputs_f64
    dtype, hh, ww, cin, cout, k = case
    print(f"\n[case] phased conv {case}", flush=True)
    sizes = dict(hh=hh, ww=ww, cin=cin, cout=cout, k=k)
    raw, x = inputs_f64("conv", dtype=dtype, **sizes)
    ref = run_unfused(OC.build("conv", **sizes), x)
    r = PlanRunner(graphs.build("conv", dtype=dtype, **sizes), "fused")
    assert "offen lds" in r.plan.kernel_source(0)
    out = r.run(raw)
    ok, mx, rel = close(out["Y"], ref["Y"], TOL[dtype])
    assert ok, f"max abs err {mx:.3e}, normwise rel {rel:.3e}"


# Waits on the oldest loads only, where loads take long and very differently:
# every shape of three or more stages over a full chip, with a contraction that
# ends inside a chunk (loads out of the buffer's range among the others), and
# padded convolutions.  A tile read before it landed changes some bytes.
def _repeat(r, what):
    from paper_2406_09465_amd._abi import lib
    r.launch_bound()
    torch.cuda.synchronize()
    first = [t.clone() for t in r.outs]
    flush = torch.empty(512 << 20, dtype=torch.uint8, device="cuda")
    stream = torch.cuda.current_stream().cuda_stream
    for i in range(60):
        for t in r.outs:
            t.zero_()
        if i >= 30:
            assert lib.korch_flush_caches(C.c_void_p(flush.data_ptr()), C.c_size_t(flush.numel()), 0, C.c_void_p(stream)) == 0
        r.launch_bound()
        torch.cuda.synchronize()
        assert all(torch.equal(a.view(torch.uint8), b.view(torch.uint8)) for a, b in zip(first, r.outs)), f"{what}: execution {i}"


@pytest.mark.gpu
@pytest.mark.parametrize("cfg", [c for c in SHAPES + F32_SHAPES if int(c.split(",")[6]) >= 3] + SPLITS + F32_SPLITS)
def test_phased_repeats_bitwise(cfg, monkeypatch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    monkeypatch.setenv("KORCH_GEMM_PHASED", cfg)
    bm, bn, ks = int(cfg.split(",")[0]), int(cfg.split(",")[1]), int((cfg.split(",") + ["1"])[7])
    dtype = "f32" if cfg in F32_SHAPES + F32_SPLITS else "bf16"
    m, n, k = 16 * bm, (16 // ks if ks > 1 else 16) * bn, 1034 * ks + (1 if dtype == "f32" else 0)
    print(f"\n[case] phased repeats {cfg} {m}x{n}x{k} {dtype}", flush=True)
    r, x = _run(m, n, k, dtype, "residual", seed=k)
    assert "offen lds" in r.plan.kernel_source(0)
    rows = slice(0, m, 61)
    full, r.outs = r.outs, [r.outs[0][rows]]
    _check(r, {nm: v[rows] if nm in ("A", "R") else v for nm, v in x.items()}, k, dtype)
    r.outs = full
    _repeat(r, cfg)


@pytest.mark.gpu
@pytest.mark.parametrize("case", [("f16", 104, 104, 128, 256, 3), ("f32", 96, 90, 64, 128, 3)], ids=lambda c: "x".join(map(str, c)))
def test_phased_convolution_repeats_bitwise(case):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2406_09465_amd import graphs
    from paper_2406_09465_amd.runner import PlanRunner
    from tests.helpers import inputs_f64
    dtype, hh, ww, cin, cout, k = case
    print(f"\n[case] phased conv repeats {case}", flush=True)
    sizes = dict(hh=hh, ww=ww, cin=cin, cout=cout, k=k)
    raw, _ = inputs_f64("conv", dtype=dtype, **sizes)
    r = PlanRunner(graphs.build("conv", dtype=dtype, **sizes), "fused")
    assert "offen lds" in r.plan.kernel_source(0)
    r.set_inputs(raw)
    r.bind()
    _repeat(r, str(case))
