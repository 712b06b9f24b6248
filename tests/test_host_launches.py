"""What the library's host code launches, on the CPU: fake_hip.cpp stands in for the HIP
runtime, with several devices, in a process of its own (no PyTorch, whose runtime would be
loaded otherwise).  Each scenario runs in a child and prints its launches."""
import ctypes as C
import json
import os
import re
import subprocess
import sys
import types

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
DOUBLES = 32            # scalars of an instance, in the order of enum Scal


class Fake:
    """The fake runtime and the library bound to it; `launches` of the calls made."""

    def __init__(self, path):
        self.hip = C.CDLL(path, mode=C.RTLD_GLOBAL)
        sys.modules["torch"] = types.ModuleType("torch")
        sys.modules["torch"].Tensor = type("Tensor", (), {})
        sys.path.insert(0, ROOT)
        import paper_1609_03488_amd as P
        self.P, self.launches, self.scalars, self.on_launch = P, [], {}, None
        with open(os.path.join(ROOT, "paper_1609_03488_amd", "csrc", "common.hpp")) as f:
            body = re.search(r"enum Scal : int \{(.*?)NSC_USED", f.read(), re.S).group(1)
        self.slot = {n: i for i, n in enumerate(re.findall(r"\bSC_[A-Z]+\b", re.sub(r"//.*", "", body)))}
        kind = C.CFUNCTYPE(None, C.c_char_p, C.POINTER(C.c_uint), C.c_size_t, C.c_int, C.POINTER(C.c_void_p))
        self._call = kind(self._launched)
        self.hip.fake_callback(self._call)
        self.hip.fake_stream.restype = C.c_void_p
        P.lib()

    def _launched(self, name, grid, lds, device, args):
        name = re.search(r"k_[a-z0-9_]+", name.decode()).group(0)
        self.launches.append(dict(name=name, grid=[grid[0], grid[1], grid[2]], lds=lds, device=device))
        if name == "k_gather_scalars":   # the instances' scalars, the same for all
            n = C.cast(args[1], C.POINTER(C.c_int))[0]
            out = C.cast(C.cast(args[2], C.POINTER(C.c_void_p))[0], C.POINTER(C.c_double))
            for i in range(n):
                for k, v in self.scalars.items():
                    out[i * DOUBLES + self.slot[k]] = v
        if self.on_launch:
            self.on_launch(self.launches[-1], args)

    def solver(self, pr, device=0, batch=1, **kw):
        """Handle of a solver whose stream is on `device`; every instance has data."""
        P, L = self.P, self.P.lib()
        st = P.Settings.make(use_graph=0, **kw)
        q = np.asarray(pr.q, dtype=np.int64)
        head = (pr.op._h, int(pr.l), q.ctypes.data_as(C.POINTER(C.c_int64)), len(q), C.byref(st))
        nb = C.c_size_t()
        assert L.cgs_workspace_bytes(*head, batch, C.byref(nb)) == 0
        buf = np.zeros(nb.value + 256, dtype=np.uint8)
        ptr = buf.ctypes.data + (-buf.ctypes.data) % 256
        h = C.c_void_p()
        rc = L.cgs_solver_create(*head, batch, ptr, nb.value, self.hip.fake_stream(device), C.byref(h))
        assert rc == 0, L.cgs_last_error()
        self.keep = getattr(self, "keep", []) + [(buf, pr)]
        b, c = (np.ascontiguousarray(v, dtype=np.float64) for v in (pr.b, pr.c))
        for i in range(batch):
            assert L.cgs_solver_set_data(h, i, b.ctypes.data_as(C.POINTER(C.c_double)),
                                         c.ctypes.data_as(C.POINTER(C.c_double))) == 0
        return h

    def deconv(self, n, k):
        return self.P.deconv_problem(np.ones(k) / k, np.ones(n + k - 1))

    def ok(self, rc):
        assert rc == 0, self.P.lib().cgs_last_error()


def lds_by_current_device(f, create, launch):
    """LDS of the fused launches of a solver on device 1, created and run while the calling
    thread's current device is `create` and `launch`."""
    f.hip.fake_set_device(int(create))
    h = f.solver(f.deconv(1700, 201), device=1, precision=f.P.FP64, fused_lone_max=0)
    f.hip.fake_set_device(int(launch))
    f.ok(f.P.lib().cgs_solver_iterate(h, 3))
    return [(v["lds"], v["device"]) for v in f.launches if v["name"] == "k_fused"]


def launches_of_creation(f, before):
    """Launches on device 0 that create an FP32 solver there, after (before = 1) one on a
    stream of device 1 was created with the same device current."""
    if int(before):
        f.solver(f.deconv(3000, 201), device=1)
        f.launches.clear()
    f.solver(f.deconv(3000, 201), device=0)
    return [(v["name"], v["grid"]) for v in f.launches if v["device"] == 0]


def steps_of_launches(f, check_every, intervals, cg_max, max_iters):
    """Steps of each fused launch of a solve that runs to its iteration limit."""
    steps = []

    def fused(launch, args):
        if launch["name"] != "k_fused":
            return
        a = C.cast(args[1], C.POINTER(C.c_int))       # FusedArgs: nsteps, check, ...
        if a[1]:
            steps.append(a[0])
            f.scalars["SC_ITER"] += a[0]
            f.scalars["SC_ACTIVE"] = 1.0 if f.scalars["SC_ITER"] < int(max_iters) else 0.0

    f.scalars = dict(SC_ACTIVE=1.0, SC_PHASE=2.0, SC_ITER=0.0)
    f.on_launch = fused
    h = f.solver(f.deconv(300, 31), check_every=int(check_every), intervals_per_sync=int(intervals),
                 cg_max_iters=int(cg_max), max_iters=int(max_iters))
    f.ok(f.P.lib().cgs_solve(h, None))
    return steps


def timed_steps(f, family, precision):
    """For each step the autotuner runs: iteration, limit and suspension flag of its last CG
    update."""
    last, steps = [], []

    def seen(launch, args):
        if launch["name"] == "k_cg_update":   # (tables, z, r, p, q, it, cg_max, gate, track, folded, last, start)
            last[:] = [C.cast(args[i], C.POINTER(C.c_int))[0] for i in (5, 6, 10)]
        if launch["name"] == "k_project":
            steps.append(list(last))

    if family == "deconv":
        pr = f.deconv(20000, 201)
    else:
        pr = f.P.lasso_problem(np.ones((40, 90)) / 40, np.ones(40), 0.1)
    h = f.solver(pr, precision=int(precision), fused_max=0, batch=3 if int(precision) == f.P.BF16 else 1)
    f.on_launch = seen
    f.ok(f.P.lib().cgs_solver_autotune(h, 2, (C.c_int32 * 4)()))
    return steps


def product_gates(f, cg_per_step):
    """Gates of the dense products of each step of a solve whose steps make cg_per_step CG
    iterations (checks left out)."""
    steps, gates = [], []

    def seen(launch, args):
        if launch["name"] == "k_gemv":      # (tables, launch, adj, out, in, base, sigma, gate, own)
            gates.append(C.cast(args[7], C.POINTER(C.c_int))[0])
        if launch["name"] == "k_project":
            steps.append(gates[-3:])
            f.scalars["SC_ITER"] += 1.0
            f.scalars["SC_CGTOT"] += float(cg_per_step)
            f.scalars["SC_ACTIVE"] = 1.0 if f.scalars["SC_ITER"] < 60 else 0.0

    pr = f.P.lasso_problem(np.ones((40, 90)) / 40, np.ones(40), 0.1)
    h = f.solver(pr, fused_max=0, cg_max_iters=1)
    f.scalars = dict(SC_ACTIVE=1.0, SC_PHASE=1.0, SC_ITER=0.0, SC_CGTOT=9.0)
    f.on_launch = seen
    f.ok(f.P.lib().cgs_solve(h, None))
    return steps


def direct_convolution(f, n, k, precision, ids):
    """Grid and LDS of the direct convolution's launch for A x."""
    n, k = int(n), int(k)
    op = f.P.Operator(n + k - 1, n).add_conv(0, 0, np.ones(k), n)
    for _ in range(int(ids)):
        op.add_identity(0, 0, 1)
    pr = types.SimpleNamespace(op=op, l=n + k - 1, q=[], b=np.ones(n + k - 1), c=np.ones(n))
    h = f.solver(pr, precision=int(precision), conv_mfma=0, fused_max=0)
    f.launches.clear()
    x, y = np.ones(n), np.ones(n + k - 1)
    f.ok(f.P.lib().cgs_solver_apply(h, 0, *(v.ctypes.data_as(C.POINTER(C.c_double)) for v in (x, y))))
    return [(v["grid"][0], v["lds"]) for v in f.launches if v["name"] == "k_conv"]


def dense_launches(f, precision, adj):
    """Launches of the dense products (name, grid, own) as an apply makes them and as the
    timing call does."""
    rec = []

    def seen(launch, args):
        own = {"k_gemv": 8, "k_gemm_reduce": 15}.get(launch["name"])
        if launch["name"] in ("k_gemv", "k_gemm_pack", "k_gemm_bf16", "k_gemm_reduce"):
            rec.append((launch["name"], launch["grid"], C.cast(args[own], C.POINTER(C.c_int))[0] if own else None))

    P, adj, dp = f.P, int(adj), C.POINTER(C.c_double)
    A = np.ones((300, 500))
    op = P.Operator(700, 900).add_identity(0, 0, 400).add_dense(30, 40, A).add_dense(350, 600, A[:200, :300])
    pr = types.SimpleNamespace(op=op, l=700, q=[], b=np.ones(700), c=np.ones(900))
    h = f.solver(pr, precision=int(precision), fused_max=0, batch=3)
    f.on_launch = seen
    x, y = np.ones(900), np.ones(700)
    x, y = (v.ctypes.data_as(dp) for v in (x, y))
    f.ok(P.lib().cgs_solver_apply(h, adj, y if adj else x, x if adj else y))
    apply = list(rec)
    rec.clear()
    f.ok(P.lib().cgs_solver_kernel_time(h, 2 + adj, 1, C.byref(C.c_double())))
    return apply, rec


def setup_launches(f, n, k, limit):
    """CG launches of the FP64 setup solve of one instance that needs no iteration."""
    f.scalars = dict(SC_ACTIVE=1.0, SC_PHASE=0.0)
    h = f.solver(f.deconv(int(n), int(k)), precision=f.P.FP64, fused_lone_max=0, setup_max_iters=int(limit))
    f.launches.clear()
    f.ok(f.P.lib().cgs_solver_iterate(h, 0))
    return sorted({v["name"] for v in f.launches} & {"k_setup_cg", "k_cg_update"})


def general_form_lds(f, attributes):
    """Dynamic LDS of the fused steps of an instance of the general form (two convolutions)
    that could use more than there is; attributes = 0: the runtime does not tell a kernel's
    attributes."""
    f.hip.fake_func_attributes(int(attributes))
    op = f.P.Operator(8000, 7000).add_conv(0, 0, np.ones(101), 3000).add_conv(4000, 3500, np.ones(31), 3000)
    pr = types.SimpleNamespace(op=op, l=8000, q=[], b=np.ones(8000), c=np.ones(7000))
    h = f.solver(pr, precision=f.P.FP64, fused_lone_max=0)
    f.launches.clear()
    f.ok(f.P.lib().cgs_solver_iterate(h, 3))
    return max(v["lds"] for v in f.launches if v["name"] == "k_fused")


def static_lds(obj, tmp):
    """Static LDS bytes of the kernels of an object file compiled for gfx950."""
    llvm = "/opt/rocm/llvm/bin/"
    fat, code = os.path.join(tmp, "fat"), os.path.join(tmp, "code")
    subprocess.run([llvm + "llvm-objcopy", f"--dump-section=.hip_fatbin={fat}", obj, os.path.join(tmp, "out")], check=True)
    subprocess.run([llvm + "clang-offload-bundler", "--unbundle", "--type=o", f"--input={fat}", f"--output={code}",
                    "--targets=hipv4-amdgcn-amd-amdhsa--gfx950"], check=True)
    notes = subprocess.run([llvm + "llvm-readelf", "--notes", code], check=True, capture_output=True, text=True).stdout
    return dict(zip(re.findall(r"^ +\.name: +_\S*?(k_[a-z_]+I?[df]?)\S*$", notes, re.M),
                    map(int, re.findall(r"\.group_segment_fixed_size: (\d+)", notes))))


def vectors_moved(f, want):
    """Vectors the device hands over for a solution call with x, y and s (bits of want)."""
    want = int(want)
    h = f.solver(f.deconv(3000, 31))
    out = [np.full(n, 7.0) for n in (3001, 6031, 6031)]
    f.launches.clear()
    f.ok(f.P.lib().cgs_solver_get_solution(h, 0, *((v.ctypes.data_as(C.POINTER(C.c_double)) if want >> i & 1 else None)
                                                   for i, v in enumerate(out))))
    assert [bool((v != 7.0).all()) for v in out] == [bool(want >> i & 1) for i in range(3)]
    return sum(v["grid"][1] for v in f.launches if v["name"].startswith("k_extract"))


SCENARIOS = {v.__name__: v for v in (vectors_moved, general_form_lds, setup_launches, dense_launches, direct_convolution, lds_by_current_device, launches_of_creation, steps_of_launches, timed_steps,
                                     product_gates)}


@pytest.fixture(scope="session")
def fake(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("fake") / "fake_hip.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    os.path.join(HERE, "fake_hip.cpp"), "-o", so], check=True)

    def run(scenario, *args):
        r = subprocess.run([sys.executable, os.path.abspath(__file__), so, scenario.__name__, *map(str, args)],
                           capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stderr
        return json.loads(r.stdout.splitlines()[-1])

    return run


# the register form of this size needs 67 KB, more than the 64 KB that need no attribute
@pytest.mark.parametrize("create,launch", [(1, 0), (0, 1), (0, 0), (2, 3)])
def test_fused_lds_is_the_handles_devices(fake, create, launch):
    """Chosen and launched by the device of the handle's stream, whatever device the calling
    thread has current."""
    want = fake(lds_by_current_device, 1, 1)
    assert want and all(lds > 65536 and dev == 1 for lds, dev in want[-1:])
    assert fake(lds_by_current_device, create, launch) == want


def test_creation_does_not_depend_on_other_devices(fake):
    """What a solver needs on its device (the FFT engine's table) is written there whichever
    devices' streams served others before."""
    alone = fake(launches_of_creation, 0)
    assert any(name == "k_conv_spectrum" for name, _ in alone)
    assert fake(launches_of_creation, 1) == alone


# the product of a round's intervals and check_every past 31 bits; the default; intervals
# longer than a launch of 16 would be; more intervals a round than a launch; long CG solves
@pytest.mark.parametrize("check_every,intervals,cg_max,max_iters,want", [
    (2 ** 28, 2, 10, 300, [300]), (10 ** 9, 2, 10, 300, [300]), (2 ** 31 - 1, 64, 10, 300, [300]),
    (10, 2, 10, 400, [160, 160, 80]), (1000, 2, 10, 4500, [1000, 1000, 1000, 1000, 500]),
    (10, 64, 10, 700, [160, 160, 160, 160, 60]), (10, 2, 10000, 40, [10, 10, 10, 10]), (1, 2, 10, 40, [16, 16, 8])])
def test_steps_of_a_fused_launch(fake, check_every, intervals, cg_max, max_iters, want):
    """At most 16 intervals and 8000 CG iterations to a launch, at least one interval."""
    assert fake(steps_of_launches, check_every, intervals, cg_max, max_iters) == want


@pytest.mark.parametrize("family,precision", [("deconv", 0), ("deconv", 1), ("dense", 0), ("dense", 1), ("dense", 2)])
def test_every_timed_step_ends_its_cg(fake, family, precision):
    """The projection reads what the update that ends CG leaves: the last update of each step
    the autotuner times is at the iteration limit or may suspend the instance."""
    steps = fake(timed_steps, family, precision)
    assert steps and all(it + 1 == limit or last for it, limit, last in steps)


# workgroups per tile of 256 (FP64) or 512 outputs, and bytes of LDS (taps and window)
@pytest.mark.parametrize("n,k,precision,ids,per,lds", [
    (5000, 33, 0, 4, 1, (2 * 36 + 264) * 8), (5000, 33, 0, 5, 2, (2 * 36 + 264) * 8),
    (5000, 124, 0, 0, 1, (2 * 124 + 264) * 8), (5000, 125, 0, 0, 2, (2 * 128 + 264) * 8),
    (130000, 257, 0, 0, 2, (2 * 260 + 264) * 8), (140000, 257, 0, 9, 1, (2 * 260 + 264) * 8),
    (140000, 2047, 0, 0, 1, (2 * 1024 + 264) * 8), (5000, 5, 1, 0, 2, (2 * 8 + 528) * 4),
    (300000, 5, 1, 0, 1, (2 * 8 + 528) * 4), (300000, 2047, 1, 9, 1, (2 * 2048 + 528) * 4)])
def test_form_of_the_direct_convolution(fake, n, k, precision, ids, per, lds):
    """Narrow form (two workgroups per tile) up to 512 tiles and from the kernel lengths or
    numbers of identity blocks where it is the faster one; the wide form's chunks of taps leave the LDS for eight waves."""
    tile = 256 if precision == 0 else 512
    assert fake(direct_convolution, n, k, precision, ids) == [[per * -(-(n + k - 1) // tile), lds]]


@pytest.mark.parametrize("precision", [0, 1, 2])
@pytest.mark.parametrize("adj", [0, 1])
def test_timed_dense_products_are_an_applys(fake, precision, adj):
    """Two dense blocks that own their ranges: the timing call launches what an apply does,
    initialisation and the written base and identity blocks included."""
    apply, timed = fake(dense_launches, precision, adj)
    assert len(apply) == (6 if precision == 2 else 2) and timed == apply
    assert all(own == 1 for _, _, own in apply if own is not None)


# 640 units and one per padded tap (28, 104, 1000) and output of a thread (2, 3, 4) an iteration
@pytest.mark.parametrize("n,k,limit,alone", [(600, 25, 500, True), (600, 25, 9195, True), (600, 25, 9196, False),
                                             (1000, 101, 6722, True), (1000, 101, 6723, False),
                                             (1000, 1000, 1379, True), (1000, 1000, 1380, False)])
def test_setup_launch_is_bounded_by_its_work(fake, n, k, limit, alone):
    """The setup solve runs in one launch where its iteration limit keeps that within 6.4
    million units (0.1 s at 16 ns), else launch by launch."""
    assert fake(setup_launches, n, k, limit) == (["k_setup_cg"] if alone else ["k_cg_update"])


@pytest.mark.parametrize("attributes", [0, 1])
def test_general_form_takes_the_lds_there_is(fake, tmp_path, attributes):
    """Static and dynamic LDS together are the workgroup's 160 KB, whether or not the runtime
    tells the kernels' attributes, and nearly all of it is dynamic."""
    obj = os.path.join(ROOT, "paper_1609_03488_amd", "_build", "fused_hip.o")
    if not os.path.exists(obj):
        pytest.skip("objects of the build are not there")
    static = static_lds(obj, str(tmp_path))
    dynamic = fake(general_form_lds, attributes)
    assert set(static) == {"k_fusedId", "k_fusedIf", "k_setup_cg"}
    assert dynamic + max(static.values()) <= 160 << 10 and dynamic >= (160 << 10) - 1024


@pytest.mark.parametrize("want", range(8))
def test_solution_moves_what_is_asked_for(fake, want):
    assert fake(vectors_moved, want) == bin(want).count("1")


G_ADMM, G_ADMM_CG = 3, 4      # enum Gate


@pytest.mark.parametrize("cg_per_step", [0, 1])
def test_idle_cg_leaves_the_products_out(fake, cg_per_step):
    """Once the host has seen a round of steps without CG iterations, the next ones gate the
    first iteration's products on the start test; with iterations it keeps them ungated."""
    steps = fake(product_gates, cg_per_step)
    assert len(steps) == 60 and all(s == [G_ADMM] * 3 for s in steps[:20])
    assert all(s == [G_ADMM] + [G_ADMM if cg_per_step else G_ADMM_CG] * 2 for s in steps[20:])


if __name__ == "__main__":
    print(json.dumps(SCENARIOS[sys.argv[2]](Fake(sys.argv[1]), *sys.argv[3:])))
