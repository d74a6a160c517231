"""Host checks of what the library launches, on the CPU: the library runs in a child process
against tests/fake_hip.cpp, which records the launches and has no device."""
import json
import os
import re
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))

PRELUDE = """
import ctypes as C, json, sys
fake = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
fake.fake_launches.restype = C.c_char_p
from paper_2108_11775_amd import _lib
lib = _lib.load()
ptr = C.c_void_p(1 << 20)  # device addresses: no kernel runs, nothing reads them
def occ(dim, M, grid=(0, 0, 0)):
    return C.byref(_lib.pdmp_occupancy(dim, M, ptr, ptr, 0.5, tuple(grid) + (0,) * (3 - len(grid))))
def stream(dev):
    return C.c_void_p(0x1000 * (dev + 1))
def launches(name, *args):
    fake.fake_launches()
    st = getattr(lib, name)(*args)
    out = []
    for line in fake.fake_launches().decode().splitlines():
        kernel, grid, block, lds = line.rsplit(" ", 3)
        out.append(dict(kernel=kernel, grid=[int(v) for v in grid[5:].split(",")],
                        block=int(block[6:]), lds=int(lds[4:])))
    assert st == 0, (st, lib.pdmp_last_error())
    return out
"""


@pytest.fixture(scope="session")
def fake_hip(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("fake") / "libfakehip.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", os.path.join(HERE, "fake_hip.cpp"),
                    "-o", lib], check=True)
    return lib


def run(fake_hip, body):
    """The JSON that `body` prints (after PRELUDE)."""
    r = subprocess.run([sys.executable, "-c", PRELUDE + body, fake_hip], capture_output=True, text=True,
                       cwd=os.path.dirname(HERE), timeout=120)
    assert r.returncode == 0, r.stderr[-2000:]
    return json.loads(r.stdout.splitlines()[-1])


def names(ls):
    return [l["kernel"].split("(")[0].split("<")[0].split("::")[-1] for l in ls]


def test_grid_check_stays_on_the_stream_s_device(fake_hip):
    """The check's blocks go with the call's launch only where the word they report to is the
    current device's; on a stream of another device the check is a launch of its own, whose
    kernel names its own device's word."""
    out = run(fake_hip, """
o = occ(2, 900, (30, 30))
calls = [("pdmp_occupancy_grad", o, ptr, 48, ptr, ptr), ("pdmp_occupancy_eval", o, ptr, 48, ptr, ptr),
         ("pdmp_morph_samples", o, None, ptr, ptr, 48, 5, 0.1),
         ("pdmp_occupancy_grad", occ(3, 4096, (16, 16, 16)), ptr, 48, ptr, ptr)]
print(json.dumps([[launches(*c, s) for s in (None, stream(0), stream(1))] for c in calls]))
""")
    for null, own, other in out:
        assert len(names(null)) == len(names(own)) == 1
        assert names(other) == ["k_grid_check"] + names(own)
        assert other[1]["grid"][0] < own[0]["grid"][0]



def test_hinges_that_fit_the_lds_are_not_split(fake_hip):
    """2-D sets of up to 5,460 hinges (64 KiB as float4 rows of three) stay in LDS over a
    morph's steps, and so do the ranges of points of a weight gradient."""
    out = run(fake_hip, """
print(json.dumps([[launches("pdmp_morph_samples", occ(2, M), None, ptr, ptr, n, 5, 0.1, None)
                   for n in (300, 8000, 40000, 1 << 21)] for M in (5441, 5460)]))
""")
    for M, calls in zip((5441, 5460), out):
        for ls in calls:
            assert names(ls) == ["k_rbf"] and ls[0]["lds"] >= (M + 3) // 4 * 48, (M, ls)
    # 1,365 chunks of points per range: 21,840 points and one hinge give ranges of a tile at most
    (ls,) = run(fake_hip, """
ws = lib.pdmp_bwd_workspace_size(2, 20000, 1365 * 4 * 60)
print(json.dumps([launches("pdmp_occupancy_bwd", occ(2, 20000), ptr, 1365 * 4 * 60, ptr, None, ptr, None,
                           ptr, ws, None)]))
""")
    rbf = [l for l in ls if names([l]) == ["k_rbf"]]
    chunks = -(-1365 * 60 // rbf[0]["grid"][1])
    assert rbf[0]["lds"] >= chunks * 48, rbf

def test_pairwise_lanes_at_the_sizes_that_lost(fake_hip):
    """The lanes per sample and threads per block where a general rule for few samples or many
    hinges loses: hinges past one tile (each block restages them in every step), fewer
    hinges than lanes, blocks that end on a nearly empty round."""
    cases = [  # dim, M, n, steps (0: values), lanes, threads
        (2, 6000, 5000, 4, 64, 512), (2, 12000, 26000, 4, 16, 512), (2, 30, 5000, 4, 8, 256),
        (3, 30, 131072, 0, 1, 256), (2, 4, 600, 4, 1, 256), (2, 2000, 26000, 0, 16, 256),
        (2, 1000, 26000, 4, 16, 256), (2, 2000, 14000, 0, 16, 512)]
    out = run(fake_hip, f"""
print(json.dumps([launches("pdmp_morph_samples", occ(d, M), None, ptr, ptr, n, T, 0.1, None) if T else
                  launches("pdmp_occupancy_eval", occ(d, M), ptr, n, ptr, ptr, None)
                  for d, M, n, T, _, _ in {cases}]))
""")
    for (d, M, n, T, lanes, threads), (l,) in zip(cases, out):
        assert l["block"] == threads and l["kernel"].startswith(f"void pdmp::k_rbf<{d}, 1, {lanes}, {threads},"), l
    (ls,) = run(fake_hip, """
ws = lib.pdmp_bwd_workspace_size(3, 1000, 200000)
print(json.dumps([launches("pdmp_occupancy_bwd", occ(3, 1000), ptr, 200000, ptr, None, ptr, None, ptr, ws,
                           None)]))
""")
    assert ls[0]["kernel"].startswith("void pdmp::k_rbf<3, 1, 1, 256,")  # one hinge per lane


def test_arm_batches_take_the_kernel_of_their_size(fake_hip):
    """One link per wave only where its rounds of 1,024 configurations are the shorter."""
    cases = [(1, 16, 10, "k_arm_grid3d"), (2, 1000, 10, "k_arm_wide"), (2, 3000, 10, "k_arm_grid3d"),
             (7, 3000, 1, "k_arm_grid3d"), (7, 3000, 10, "k_arm_wide"), (7, 4000, 10, "k_arm_grid3d")]
    out = run(fake_hip, f"""
def arm(n):
    a = _lib.pdmp_arm()
    a.n_dof, a.pts_per_link = n, 8
    return C.byref(a)
print(json.dumps([launches("pdmp_morph_samples", occ(3, 4096, (16, 16, 16)), arm(d), ptr, ptr, n, T, 0.1, None)
                  for d, n, T, _ in {cases}]))
""")
    for (d, n, T, kernel), ls in zip(cases, out):
        assert names(ls)[-1] == kernel, (d, n, T, names(ls))


MLP = """
def mlp(n_in, H, L):
    return C.byref(_lib.pdmp_mlp(n_in, H, L, ptr, ptr))
def least(n_in, H, L, B):
    # two vectors' buffers, 2,048 samples per partial row, column sums, the loss's partial sums
    al = lambda b: (b + 255) // 256 * 256
    w, S = max(H, n_in), min(max(B // 2048, 1), 64)
    return (2 * al(2 * B * w) + al(4 * S * w * w) + al(4 * w * (-(-B // 256))) + al(8192),
            al(2 * B * n_in) + 2 * al(2 * B * H))
"""


def test_mlp_workspace_never_shrinks_with_the_batch(fake_hip):
    """A workspace for the largest batch serves every smaller one."""
    out = run(fake_hip, MLP + """
Bs = sorted({b + d for b in (1, 64, 128, 256, 2048, 4096, 10240, 12288, 65536, 131072, 1 << 20)
             for d in (-1, 0, 1, 64, 65) if b + d > 0})
print(json.dumps([[lib.pdmp_mlp_workspace_size(mlp(n, H, L), B) for B in Bs]
                  for n in (1, 7, 16) for H in (1, 9, 32, 100, 128, 256, 288, 512, 600, 1024)
                  for L in (1, 3, 6)]))
""")
    for sizes in out:
        assert all(a <= b for a, b in zip(sizes, sizes[1:])), sizes


def test_mlp_workspace_of_two_buffers_is_enough(fake_hip):
    """The inference forward, the backward and the amortised morph in a workspace of two layers'
    activations or vectors."""
    out = run(fake_hip, MLP + """
res = []
for n, H, L in ((7, 16, 1), (7, 32, 3), (16, 33, 2), (6, 64, 6), (7, 100, 3), (7, 256, 3), (7, 300, 2), (5, 512, 6),
                (7, 1001, 2), (7, 1024, 6)):
    for B in (1, 31, 64, 127, 129, 700, 4095, 4096, 4097, 10001, 65535, 65536, 300007):
        m = mlp(n, H, L)
        bwd, fwd = least(n, H, L, B)
        arm = _lib.pdmp_arm()
        arm.n_dof, arm.pts_per_link = n, 8
        calls = [("pdmp_mlp_forward", m, ptr, B, ptr, None, ptr, fwd, None),
                 ("pdmp_mlp_backward", m, ptr, ptr, B, ptr, ptr, ptr, ptr, bwd, None),
                 ("pdmp_mlp_backward_weighted", m, ptr, ptr, B, ptr, 2.0, ptr, ptr, ptr, ptr, bwd, None)]
        if n <= 8:
            am = lib.pdmp_amortised_workspace_size(m, C.byref(arm), B)
            al = lambda b: (b + 255) // 256 * 256
            am -= 2 * (al(2 * B * ((H + 7) // 8 * 8)) - al(2 * B * H))
            q = C.c_void_p(2 << 20)
            calls.append(("pdmp_amortised_morph", m, occ(3, 4096, (16, 16, 16)), C.byref(arm), ptr, q, B, 5, 0.1,
                          0.5, None, None, ptr, am, None))
        for c in calls:
            fake.fake_launches()
            st = getattr(lib, c[0])(*c[1:])
            res.append((c[0], n, H, L, B, st, len(fake.fake_launches())))
print(json.dumps(res))
""")
    for r in out:
        assert r[5] == 0 and r[6] > 0, r


def test_mlp_weight_gradient_sums_at_most_2048_samples_in_fp32(fake_hip):
    """A partial row of a weight gradient is one FP32 accumulator's sum: of 2,048 samples, as far as
    64 rows go, whatever the width and depth."""
    cases = [(H, L, B) for H, L in ((64, 1), (256, 3), (256, 6), (300, 6), (512, 2), (1024, 6))
             for B in (65536, 131072, 1 << 20)]
    out = run(fake_hip, MLP + f"""
print(json.dumps([launches("pdmp_mlp_backward", mlp(7, H, L), ptr, ptr, B, ptr, ptr, ptr, ptr,
                           lib.pdmp_mlp_workspace_size(mlp(7, H, L), B), None) for H, L, B in {cases}]))
""")
    for (H, L, B), ls in zip(cases, out):
        widths = [7] + [H] * L + [7]
        tiles = [-(-a // 128) * -(-b // 128) for a, b in zip(widths, widths[1:])]
        wg = [l["grid"][0] for l, k in zip(ls, names(ls)) if k == "k_mlp_wgrad"]
        if len(wg) == 1:
            tiles = [sum(tiles)]
        for blocks, t in zip(wg, reversed(tiles)):
            assert blocks // t >= min(64, B // 2048), (H, L, B, blocks, t)


def test_layered_products_keep_their_waves():
    """The tiled GEMM of the widths without a fused kernel lives off eight waves per SIMD: at
    most 64 registers (5 waves: 20 to 30 % slower forwards from 65,536 samples on)."""
    readelf = "/opt/rocm/llvm/bin/llvm-readelf"
    if not os.path.exists(readelf):
        pytest.skip("no llvm-readelf")
    from paper_2108_11775_amd import _lib
    data = open(_lib.LIB_PATH, "rb").read()
    found, at = [], data.find(b"\x7fELF", 1)
    while at >= 0:
        if data[at + 18:at + 20] == b"\xe0\x00":  # EM_AMDGPU
            r = subprocess.run([readelf, "--notes", "-"], input=data[at:], capture_output=True)
            text = r.stdout.decode(errors="replace")
            for k in re.split(r"\n\s+- \.agpr_count", text):
                m = re.search(r"\.name:\s+(\S*k_gemm\S*)", k)
                if m:
                    found.append((m[1], int(re.search(r"\.vgpr_count:\s+(\d+)", k)[1])))
        at = data.find(b"\x7fELF", at + 4)
    assert len(found) == 3 and all(v <= 64 for _, v in found), found


def kernel_registers(pattern):
    """{name: VGPRs} of the library's kernels that match `pattern`."""
    readelf = "/opt/rocm/llvm/bin/llvm-readelf"
    if not os.path.exists(readelf):
        pytest.skip("no llvm-readelf")
    from paper_2108_11775_amd import _lib
    data = open(_lib.LIB_PATH, "rb").read()
    found, at = {}, data.find(b"\x7fELF", 1)
    while at >= 0:
        if data[at + 18:at + 20] == b"\xe0\x00":  # EM_AMDGPU
            r = subprocess.run([readelf, "--notes", "-"], input=data[at:], capture_output=True)
            for k in re.split(r"\n\s+- \.agpr_count", r.stdout.decode(errors="replace")):
                m = re.search(r"\.name:\s+(\S*%s\S*)" % pattern, k)
                if m:
                    found[m[1]] = int(re.search(r"\.vgpr_count:\s+(\d+)", k)[1])
        at = data.find(b"\x7fELF", at + 4)
    return found


@pytest.mark.parametrize("mode,most", [(4, 168), (5, 128)])
def test_2d_inverse_kernels_keep_their_waves(mode, most):
    """A grid of at most 32 hinges in y: three waves per SIMD with the log-determinant (mode 4),
    four in the inverse (5); a wave less cost 10 to 28 % from 131,072 samples on."""
    regs = kernel_registers(r"k_grid2d_invILi1ELi[1-4]ELi%dE" % mode)
    assert len(regs) == 4 and max(regs.values()) <= most, regs


def test_tanh_net_of_one_hidden_layer_sums_in_the_lds(tmp_path):
    """No products to wait for: the lanes' sums by row swaps, on the busy vector unit, cost 3 to
    6 % from 33,000 points on."""
    objdump = "/opt/rocm/llvm/bin/llvm-objdump"
    if not os.path.exists(objdump):
        pytest.skip("no llvm-objdump")
    from paper_2108_11775_amd import _lib
    data = open(_lib.LIB_PATH, "rb").read()
    seen, name, at = {}, "", data.find(b"\x7fELF", 1)
    while at >= 0:
        if data[at + 18:at + 20] == b"\xe0\x00":  # EM_AMDGPU
            (tmp_path / "co").write_bytes(data[at:])
            r = subprocess.run([objdump, "-d", str(tmp_path / "co")], capture_output=True)
            for line in r.stdout.decode(errors="replace").splitlines():
                m = re.match(r"[0-9a-f]+ <(.*)>:", line)
                name = m[1] if m else name
                if "k_tanh_netILi" in name and ("_bpermute" in line or "v_permlane" in line):
                    seen.setdefault(name, set()).add("swap" if "v_permlane" in line else "lds")
        at = data.find(b"\x7fELF", at + 4)
    one = {k: v for k, v in seen.items() if re.search(r"ILi[23]ELi[124]ELi1E", k)}
    assert len(one) == 18 and all(v == {"lds"} for v in one.values()), one


@pytest.mark.parametrize("device", [None, 1, "cuda:1", "cuda"])
def test_sync_takes_a_device_as_torch_names_it(monkeypatch, device):
    import types

    import torch

    import paper_2108_11775_amd as P
    seen = []
    monkeypatch.setattr(torch.cuda, "current_stream",
                        lambda d=None: types.SimpleNamespace(cuda_stream=("stream of", d)))
    monkeypatch.setattr(P._lib, "call", lambda *a: seen.append(a))
    P.sync(device)
    assert seen == [("pdmp_sync", ("stream of", device))]
