"""Host-side checks of the C-ABI library that need no GPU: it loads, exports
every symbol the header declares, sizes workspaces, and rejects bad input
before touching the device."""
import ctypes as C
import os
import re
import struct
import subprocess

import pytest

from paper_2104_06272_amd import binding, build, workloads as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(binding.LIB_PATH):
        build.build(verbose=False)
    return binding.load()


def test_exports_match_header(lib):
    text = open(os.path.join(ROOT, "include", "anakin.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    declared = set(re.findall(r"\b(anakin_[a-z_]+)\s*\(", text))
    assert declared == set(binding.EXPORTS)
    for name in declared:
        assert hasattr(lib, name), name


def test_workspace_sizes(lib):
    sizes = {n: binding.workspace_bytes(W.get(n)) for n in W.ORDER}
    for n, s in sizes.items():
        assert s > 0 and s % 256 == 0, n
    assert sizes["catch_small"] < sizes["catch_4096"] < sizes["maze_16384"]
    assert sizes["maze_16384"] < 64 << 30               # far inside one GPU's 288 GB
    small = W.get("catch_small")
    assert binding.workspace_bytes(small, B=128) > binding.workspace_bytes(small, B=64)


@pytest.mark.parametrize("mutate", [
    lambda c: c.update(B=60),                                   # not a multiple of 16
    lambda c: c.update(B=0),
    lambda c: c.update(T=0),
    lambda c: c["net"].update(hidden=[48]),                     # not a power of two
    lambda c: c["net"].update(hidden=[16]),
    lambda c: c["net"].update(hidden=[64] * 5),
    lambda c: c["net"].update(policy="tanh_gaussian"),          # wrong policy for catch
    lambda c: c["net"].update(lr=0.0),
    lambda c: c["env"].update(rows=1),
    lambda c: c.update(env=dict(kind="maze", rows=32, cols=32, max_steps=10, p_wall=0.2)),
    # no acting tile fits: a 32-wide layer needs tiles of 32 envs (B = 48 is not a multiple), and a 1024-wide last
    # layer with the only tile it allows (16 envs) is 2 KB over the LDS of a workgroup
    lambda c: (c.update(B=48), c["net"].update(hidden=[32, 64])),
    lambda c: (c.update(B=16), c["net"].update(hidden=[1024])),
    lambda c: (c.update(B=16), c["net"].update(hidden=[1024, 1024])),
])
def test_bad_configs_are_rejected_on_the_host(lib, mutate):
    cfg = W.get("catch_small")
    cfg["env"] = dict(cfg["env"])
    mutate(cfg)
    if len(cfg["net"]["hidden"]) > 4:
        cfg["net"]["hidden"] = cfg["net"]["hidden"][:4]
        env, net = binding.make_cfgs(cfg)
        net.n_hidden = 5
    else:
        env, net = binding.make_cfgs(cfg)
    assert lib.anakin_workspace_bytes(C.byref(env), C.byref(net), cfg["B"], cfg["T"]) == 0
    h = C.c_void_p()
    rc = lib.anakin_create(C.byref(h), C.byref(env), C.byref(net), cfg["B"], cfg["T"], 0, None, 0, None)
    assert rc == binding.E_BAD_CONFIG and not h.value
    assert len(lib.anakin_last_error(None)) > 0


def test_create_checks_workspace_before_any_device_call(lib):
    cfg = W.get("catch_small")
    env, net = binding.make_cfgs(cfg)
    h = C.c_void_p()
    assert lib.anakin_create(C.byref(h), C.byref(env), C.byref(net), 64, 20, 0, None, 0, None) == binding.E_INVALID_ARG
    assert lib.anakin_create(C.byref(h), C.byref(env), C.byref(net), 64, 20, 0, C.c_void_p(0x1001), 1 << 30, None) == binding.E_MISALIGNED
    assert lib.anakin_create(C.byref(h), C.byref(env), C.byref(net), 64, 20, 0, C.c_void_p(0x1000), 4096, None) == binding.E_WORKSPACE_TOO_SMALL
    assert b"need" in lib.anakin_last_error(None)
    assert lib.anakin_create(None, C.byref(env), C.byref(net), 64, 20, 0, None, 0, None) == binding.E_INVALID_ARG
    for fn in (lib.anakin_rollout, lib.anakin_learn, lib.anakin_learn_static, lib.anakin_step, lib.anakin_destroy):
        assert fn(None) == binding.E_INVALID_ARG


def test_no_gpu_means_error_not_fallback():
    import torch
    if torch.cuda.is_available():
        pytest.skip("a GPU is present")
    with pytest.raises(RuntimeError):
        binding.Anakin(W.get("catch_small"))


def build_host_program(name, tmp_path):
    """tests/host/<name>.hip: the library's host code on configurations without a device"""
    exe = str(tmp_path / name)
    where = os.path.dirname(binding.LIB_PATH)
    cmd = [build.HIPCC, *build.FLAGS, "-O1", os.path.join(ROOT, "tests", "host", name + ".hip"), "-o", exe, "-no-hip-rt",
           "-L" + where, "-Wl,-rpath," + where, "-l:" + os.path.basename(binding.LIB_PATH)]
    torch_lib = build.torch_lib_dir()
    cmd += ["-L" + torch_lib, "-Wl,-rpath," + torch_lib] if torch_lib else []
    subprocess.run(cmd + ["-L/opt/rocm/lib", "-Wl,-rpath,/opt/rocm/lib", "-lamdhip64"], check=True, stderr=subprocess.DEVNULL)
    return exe


def test_every_divisor_of_the_unroll_is_accepted_as_updates(lib, tmp_path):
    """Chunk plans of several updates per unroll, over shapes of all kinds: a divisor of T is taken, its partial sums fit
    the full unroll's room and no workgroup is without samples."""
    out = subprocess.run([build_host_program("updates_plan", tmp_path), "7", "50000"], capture_output=True, text=True)
    assert out.returncode == 0 and out.stdout.startswith("ok "), out.stdout + out.stderr


def test_update_routes(lib, tmp_path):
    """Which launches an update takes on both sides of a rule, and the scratch it asks for."""
    out = subprocess.run([build_host_program("update_routes", tmp_path)], capture_output=True, text=True)
    assert out.returncode == 0 and out.stdout == "ok\n", out.stdout + out.stderr


def test_waits_of_the_256_wide_bf16_products_cover_what_is_read(tmp_path):
    """Every form of backward_bf16.hip, in the order in which a wavefront issues its loads and stores: what a stage reads from
    LDS is older than what the wait in front of it leaves in flight."""
    exe = str(tmp_path / "order")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-O1", os.path.join(ROOT, "tests", "host", "backward_bf16_order.cpp"), "-o", exe], check=True)
    out = subprocess.run([exe], capture_output=True, text=True)
    assert out.returncode == 0 and out.stdout == "ok 12\n", out.stdout + out.stderr


def test_backward_products_keep_their_registers(lib):
    """No kernel of the backward products of whole tiles has scratch memory: backward_bf16 counts its loads and stores by hand and
    would not count those, and the split products have no register to spare."""
    image = open(binding.LIB_PATH, "rb").read()
    sizes = {}
    for entry in re.finditer(rb"\xa5\.name\xd9.(\w+)\xbb\.private_segment_fixed_size(.)", image, re.S):
        name, first = entry.group(1).decode(), entry.group(2)[0]  # (a number up to 127 is its own byte, larger ones begin with 0xcc and up)
        if "gemm_tn_nt_split" in name or "13backward_bf16" in name:
            sizes[name] = first
    assert sum("13backward_bf16" in n for n in sizes) == 8 and sum("gemm_tn_nt_split" in n for n in sizes) >= 64, len(sizes)
    assert not any(sizes.values()), {n: v for n, v in sizes.items() if v}


def test_gpu_tests_reach_every_form_of_the_split_products(lib, tmp_path):
    """The shapes of the GPU tests that hold the products on split operands to binary32 run every form of the kernel that any
    shape runs, so that a threshold that moves does not leave one untested."""
    import itertools
    import test_gpu_shapes as G
    exe = build_host_program("split_tiles", tmp_path)
    large = G.BOARDS[-1]
    assert large["rows"] * large["cols"] > 64                    # (such a board is not folded into the products)
    env = {"catch_4096": "0 {} 10 5", "pendulum_8192": "1 {} 0 0", "large": f"0 {{}} {large['rows']} {large['cols']}", "maze": "2 {} 5 7"}

    def forms(shapes):
        lines = [" ".join([env[name].format(bf16), str(B), str(T)] + [str(h) for h in hidden]) for name, hidden, B, T, bf16 in shapes]
        out = subprocess.run([exe], input="\n".join(lines), capture_output=True, text=True, check=True).stdout.splitlines()
        assert len(out) == len(lines)
        return [set(line.split()) if not line.startswith("refused") else set() for line in out]

    every = set().union(*forms([(name, hidden, B, T, 0) for name in env for B, T in ((16, 3), (64, 63), (2064, 17), (16384, 20)) for n in (2, 3)
                                for hidden in itertools.product([32, 64, 128, 256, 512, 1024], repeat=n)]))
    tested = set().union(*forms([(name, hidden, B, T, 0) for name, hidden in G.SPLIT_FORMS + [("catch_4096", h) for h in G.SPLIT_PAIRS] +
                                 [("large", h) for h in G.SPLIT_LAYERS] + [("maze", h) for h in G.SPLIT_PAIRS] for B, T in G.SPLIT_BATCHES]))
    assert tested == every, every ^ tested
    assert len(every) == 77, len(every)
    # the bf16 nets: every pairing of large tiles that widths of 128 and more can have
    large = [f for s in G.SPLIT_LARGE_BF16 for f in forms([s + (2064, 17, 1)])[0]]
    assert {f.split(":")[1] for f in large} >= {"256x256/256", "128x128/256", "128x128/128"} and all(f.startswith("many:") for f in large)


def registers_per_lane(pattern, tmp_path):
    """{kernel: vector registers} of the library's own code objects, kernels whose mangled name matches `pattern`"""
    image, magic, out = open(binding.LIB_PATH, "rb").read(), b"__CLANG_OFFLOAD_BUNDLE__", {}
    for at in (m.start() for m in re.finditer(magic, image)):
        (n,), pos = struct.unpack_from("<Q", image, at + len(magic)), at + len(magic) + 8
        for _ in range(n):
            offset, size, length = struct.unpack_from("<QQQ", image, pos)
            triple, pos = image[pos + 24:pos + 24 + length], pos + 24 + length
            if not triple.endswith(b"gfx950") or not size:
                continue
            obj = tmp_path / "code.o"
            obj.write_bytes(image[at + offset:at + offset + size])
            notes = subprocess.run([os.path.join(os.path.dirname(build.HIPCC), "..", "llvm", "bin", "llvm-readelf"), "--notes", str(obj)],
                                   capture_output=True, text=True, check=True).stdout
            for name, count in re.findall(r"\.name: +(_Z\S+)\n(?:(?!\.name: +_Z).)*?\.vgpr_count: +(\d+)", notes, re.S):
                if re.search(pattern, name):
                    out[name] = int(count)
    return out


def test_actor_of_128_units_holds_registers_only_beside_a_learner(lib, tmp_path):
    """Two workgroups of the 128-wide actor of boards share a compute unit (eight wavefronts each: 128 registers); the form
    that runs beside a learner's replay keeps that out with more."""
    plain = registers_per_lane(r"rollout_resident_kernelILi[02]ELi128ELi[12]ELb0E", tmp_path)
    beside = registers_per_lane(r"rollout_resident_kernelILi[02]ELi128ELi[12]ELb1E", tmp_path)
    assert len(plain) == 4 and max(plain.values()) <= 128, plain
    assert len(beside) == 4 and min(beside.values()) >= 160, beside


def test_bench_models_the_bf16_products_that_share_a_launch():
    """bench.py's work per launch: bf16 layers with a 128-wide side are in the shared launch, at bf16 rates, and the other
    layers in launches of their own; an fp32 net of the same widths is all split products."""
    import bench
    cfg = W.get("pendulum_8192")
    cfg["net"] = dict(cfg["net"], hidden=[512, 512, 128], dtype="bf16")
    M = cfg["B"] * cfg["T"]
    models, _ = bench.kernel_models(cfg, 1, launched=("gemm_tn", "gemm_nt_mask", "gemm_tn_nt"))
    assert models["gemm_tn_nt"] == ("hbm", 2.0 * (2 * 512 + 128) * M / 1e9, bench.PEAK_HBM_GBS, "GB/s")
    assert models["gemm_tn"] == ("hbm", 2.0 * (512 + 512) * M / 1e9, bench.PEAK_HBM_GBS, "GB/s")
    assert models["gemm_nt_mask"] == ("hbm", (2.0 * 512 + 512 / 4 + 2.0 * 512) * M / 1e9, bench.PEAK_HBM_GBS, "GB/s")
    cfg["net"]["dtype"] = "fp32"
    models, _ = bench.kernel_models(cfg, 1, launched=("gemm_tn_nt",))
    assert models["gemm_tn_nt"] == ("mfma", 4.0 * (512 * 512 + 512 * 128) * M / 1e12, bench.PEAK_SPLIT_TFLOPS, "TFLOP/s")
