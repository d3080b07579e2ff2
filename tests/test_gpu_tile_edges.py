"""GPU parity at the edges of tiles, key groups and dispatch rules, against the fp64 oracle.

Tolerances are the ones of the other parity tests (parity.py's compare): bf16 outputs 2e-2
and fp32 outputs 1e-5 of a row's norm, selections exact outside the stated bands."""

import numpy as np
import pytest
import torch

import oracle
from parity import compare, dims_of, gpu_outputs, run_oracle, to_device
from synth import WORKLOADS, make_case, make_memory_case, make_output_grad

pytestmark = pytest.mark.gpu

H_TOL = {"f32": 1e-5, "bf16": 2e-2}


@pytest.fixture(scope="module")
def lib():
    import paper_2608_22883_amd as lib

    assert torch.cuda.is_available()
    return lib


def _wl(dtype, **kw):
    base = WORKLOADS["tiny_f32"] if dtype == "f32" else WORKLOADS["llava_b1"].with_(d=512, d_m=256)
    return base.with_(**kw)


def _run(lib, case):
    wl = case.workload
    fv = lib.Fovea(dims_of(wl, case.weights, 1 if wl.dtype == "bf16" else 0), case.weights, device="cuda")
    print(f"[gpu] edges {wl.dtype}: B={wl.B} n={case.n_nodes} d={wl.d} d_m={wl.d_m} d_c={wl.d_c} "
          f"m_max={case.m_max} k_max={case.k_max}", flush=True)
    out = fv.retrieve_fuse(to_device(case, wl.dtype))
    torch.cuda.synchronize()
    st, bits = lib.fovea_last_error(fv.ctx)
    g = gpu_outputs(out)
    fv.close()
    assert st == 0, f"data error bits {bits:#x}"
    return g


# one key per thread and slot group (1024), each register count's last size and the next
# (2048, 4096, 8192), rows of scores that are not 16-byte aligned, k_max at both ends, masks
@pytest.mark.parametrize("dtype,M,k_max,valid", [
    ("bf16", 1025, 64, 1.0), ("bf16", 2048, 1, 0.9), ("bf16", 2050, 300, 1.0), ("f32", 4096, 64, 0.7),
    ("bf16", 4099, 128, 0.5), ("bf16", 8192, 1024, 1.0), ("f32", 8195, 256, 0.9),
    ("bf16", 16384, 256, 0.02), ("f32", 700, 1024, 0.9),
    # lists too long to rank (k_max near the number of key groups): a closer bound first
    ("bf16", 1500, 1024, 1.0), ("f32", 2048, 700, 1.0), ("bf16", 3000, 512, 0.9), ("f32", 1100, 513, 1.0)])
def test_block_selection_sizes(lib, dtype, M, k_max, valid):
    wl = _wl(dtype, B=1, T=7, M=M, k_max=k_max, tau=0.9, key_scale=(25.0, 25.0), valid_frac=valid)
    case = make_case(wl, affine="unit")
    compare(case, _run(lib, case), run_oracle(case), H_TOL[dtype], label=f"block selection {dtype} M={M}")


@pytest.mark.parametrize("dtype,M", [("f32", 5000), ("bf16", 5000), ("bf16", 1500)])
def test_block_selection_overflowing_list(lib, dtype, M):
    """Every score equal over all entries: the list of keys that reach the bound would hold
    them all (5000 do not fit it, 1500 would take longer to rank than a search), so the
    threshold is searched and its ties cut by index; and one request whose 200 best entries
    are neighbours, so that they fill few of the block's key groups."""
    wl = _wl(dtype, B=2, T=5, M=M, k_max=100, tau=0.5, key_scale=(20.0, 20.0))
    case = make_case(wl, affine="random")
    keys = case.keys.copy()
    keys[:M] = keys[0]
    keys[M:M + 200] *= 4.0
    case.keys = keys
    case.tau = np.array([0.0101, 0.9]).astype(np.float32).astype(np.float64)
    g, ref = _run(lib, case), run_oracle(case)
    compare(case, g, ref, H_TOL[dtype], label=f"block selection ties {dtype} M={M}")
    for node in range(5):
        K = int(ref["K"][node])
        assert g["K"][node] == K and g["idx"][node, :K].tolist() == list(range(K))


# few nodes: 32- and 64-row tiles of the correction layers, the row partials' limit
# (d / 16 <= d_c holds at 1024 / 64, not at 2048 / 64), layers 1 and 2 past their widest k
@pytest.mark.parametrize("T,d,d_m,d_c", [(1, 512, 256, 512), (33, 1024, 64, 64), (64, 2048, 192, 64),
                                         (64, 512, 2112, 128), (65, 512, 256, 512),
                                         (61, 256, 64, 1024), (61, 256, 64, 1088)])
def test_few_nodes(lib, T, d, d_m, d_c):
    wl = _wl("bf16", B=1, T=T, M=100, d=d, d_m=d_m, d_c=d_c, k_max=16, key_scale=(30.0, 30.0))
    case = make_case(wl, affine="unit")
    compare(case, _run(lib, case), run_oracle(case), H_TOL["bf16"], label=f"few nodes T={T} d={d} d_m={d_m}")


# whole 64-row tiles of the hidden-state GEMM (12 x 15 tiles), the last row tile ragged; the
# three-plane fp32 core in 128- and 64-row tiles
@pytest.mark.parametrize("dtype,B,T,d,d_m,d_c", [("bf16", 12, 59, 512, 896, 512), ("f32", 3, 60, 320, 192, 128),
                                                 ("f32", 1, 65, 1024, 128, 512)])
def test_batches_between_tiles(lib, dtype, B, T, d, d_m, d_c):
    wl = _wl(dtype, B=B, T=T, M=90, d=d, d_m=d_m, d_c=d_c, k_max=16, key_scale=(30.0, 30.0))
    case = make_case(wl, affine="unit")
    compare(case, _run(lib, case), run_oracle(case), H_TOL[dtype], label=f"batch {dtype} n={B * T}")


# scores: runs of 128-key tiles (a ragged last run, unaligned score rows, two chunks of nodes,
# runs shorter than the longest memory asks for), 80-key tiles (two node
# chunks, more and fewer chunks of k than stages, ragged memories), the register kernel's 64-, 80-
# and 96-key tiles, each key count of the fp32 tiles and the fp32 kernel for few nodes (whole and
# partial blocks of 16 nodes, two chunks)
@pytest.mark.parametrize("dtype,B,T,M,M_lo,d_m", [
    ("bf16", 8, 65, 6001, None, 64), ("bf16", 8, 65, 6001, None, 320), ("bf16", 4, 65, 16001, 8000, 128),
    ("bf16", 16, 66, 1999, None, 64), ("bf16", 16, 3, 1999, 5, 192), ("f32", 1, 3, 90, None, 64),
    ("f32", 5, 65, 1400, None, 64), ("f32", 12, 3, 1201, None, 192), ("f32", 16, 17, 1300, 700, 64),
    ("f32", 20, 5, 1500, None, 128), ("bf16", 4, 33, 16001, None, 256), ("bf16", 16, 17, 1000, None, 256),
    ("bf16", 34, 5, 601, None, 512), ("bf16", 32, 9, 600, None, 768), ("f32", 8, 17, 1030, None, 64),
    ("f32", 8, 70, 1030, 500, 64), ("f32", 8, 33, 1030, None, 512), ("f32", 8, 32, 1030, None, 512),
    ("bf16", 4, 66, 5301, None, 768), ("bf16", 8, 48, 11001, 500, 768)])
def test_score_tiles(lib, dtype, B, T, M, M_lo, d_m):
    wl = _wl(dtype, B=B, T=T, M=M, d_m=d_m, k_max=16, key_scale=(30.0, 30.0), **({"M_lo": M_lo} if M_lo else {}))
    case = make_case(wl, affine="unit")
    compare(case, _run(lib, case), run_oracle(case), H_TOL[dtype], label=f"scores {dtype} B={B} T={T} M={M} d_m={d_m}")


# memory builds: 64- and 128-row tiles of 128 columns, the ping-pong core's 128-, 192- and
# 256-row tiles with ragged last tiles, fp32's two heights
@pytest.mark.parametrize("dtype,rows,d_m", [("bf16", 65, 64), ("bf16", 1024, 1024), ("bf16", 2049, 1024),
                                            ("bf16", 6200, 448), ("bf16", 8300, 512), ("bf16", 2200, 512),
                                            ("bf16", 7000, 1024), ("f32", 63, 64),
                                            ("f32", 2100, 1024)])
def test_memory_build_tiles(lib, dtype, rows, d_m):
    wl = _wl(dtype, d=192, d_m=d_m)
    V, W = make_memory_case(wl, rows, affine="random")
    fv = lib.Fovea(dims_of(wl, W, 1 if dtype == "bf16" else 0), W, device="cuda")
    print(f"[gpu] build {dtype} rows={rows} d_m={d_m}", flush=True)
    keys, values = fv.build_memory(torch.tensor(V, dtype=torch.bfloat16 if dtype == "bf16" else torch.float32,
                                                device="cuda"))
    torch.cuda.synchronize()
    fv.close()
    ref = oracle.build_memory(V, W["mem_ln_g"], W["mem_ln_b"], W["W_K"], W["W_U"], W["ln_eps"],
                              gain_rounding="bf16" if dtype == "bf16" else None)
    for got, want in zip((keys, values), ref):
        got = got.double().cpu().numpy()
        rel = np.linalg.norm(got - want, axis=1) / np.linalg.norm(want, axis=1)
        assert rel.max() <= H_TOL[dtype], rel.max()


def test_backward_wide_rows_and_long_node_lists(lib):
    """Rows wider than the row kernels hold in registers, more nodes than one ballot lists,
    entries selected by none, some and many of them."""
    wl = WORKLOADS["tiny_f32"].with_(B=2, T=130, M=70, d=8256, d_m=320, d_c=64, k_max=5, k_min=5)
    case = make_case(wl, affine="random")
    W = case.weights
    f = oracle.retrieve_fuse(W, case.mem_off, case.keys, case.values, case.valid, case.node_off, case.h,
                             case.depth, case.tau, case.k_min, case.k_max)
    dh_hat = make_output_grad(case.n_nodes, wl.d, 3)
    ref = oracle.retrieve_fuse_backward(W, case.mem_off, case.keys, case.values, case.node_off, case.h,
                                        case.depth, f["idx"], f["K"], dh_hat)
    fv = lib.Fovea(dims_of(wl, W, 0), W, device="cuda")
    dev = dict(device="cuda")
    print(f"[gpu] backward edges n={case.n_nodes} d={wl.d}", flush=True)
    g = fv.retrieve_fuse_backward(to_device(case, "f32"), torch.tensor(f["K"], dtype=torch.int32, **dev),
                                  torch.tensor(f["idx"], dtype=torch.int32, **dev),
                                  torch.tensor(dh_hat, dtype=torch.float32, **dev))
    torch.cuda.synchronize()
    assert lib.fovea_last_error(fv.ctx)[0] == 0
    fv.close()
    for k, want in ref.items():
        if k not in g or want is None:
            continue
        got = g[k].double().cpu().numpy().reshape(np.shape(want))
        scale = max(float(np.abs(want).max()), 1e-30)
        # two-plane products: 2^-16 of the operands; 2e-4 as in the other backward tests
        assert float(np.abs(got - want).max()) / scale <= 2e-4, k


# a batch in which one request has most of the nodes, so that a block walks several chunks of
# 64 of them (every score kernel: 16- to 128-key tiles, both dtypes, widths with and without a
# fixed chunk count), under the tight bound on a request's nodes and under the loosest
@pytest.mark.parametrize("dtype,B,big,M,d_m", [
    ("bf16", 300, 300, 576, 256), ("bf16", 300, 700, 100, 512), ("bf16", 260, 200, 200, 320),
    ("bf16", 20, 1500, 100, 192), ("bf16", 2, 1100, 300, 1024), ("bf16", 40, 3000, 700, 768),
    ("f32", 300, 300, 576, 128), ("f32", 300, 700, 60, 64), ("f32", 16, 1500, 700, 512)])
def test_uneven_requests(lib, dtype, B, big, M, d_m):
    wl = _wl(dtype, B=B, T=1, M=M, d=256 if dtype == "bf16" else 128, d_m=d_m, d_c=64, k_max=16,
             key_scale=(30.0, 30.0))
    extra = -(-(big + B - 1) // B)
    case = make_case(wl.with_(T=extra), affine="unit")
    n = case.n_nodes
    sizes = np.ones(B, np.int64)
    sizes[B // 2] = n - (B - 1)
    case.node_off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    fv = lib.Fovea(dims_of(wl, case.weights, 1 if dtype == "bf16" else 0), case.weights, device="cuda")
    inp = to_device(case, dtype)
    got = []
    for t_max in (int(sizes.max()), n, 1 << 30):
        inp["t_max"] = t_max
        print(f"[gpu] uneven {dtype} B={B} n={n} M={M} d_m={d_m} t_max={t_max}", flush=True)
        out = fv.retrieve_fuse(inp)
        torch.cuda.synchronize()
        got.append(gpu_outputs(out))
        assert lib.fovea_last_error(fv.ctx)[0] == 0
    fv.close()
    for g in got[1:]:
        for k in g:
            assert np.array_equal(g[k], got[0][k]), k
    pick = np.r_[0:B // 2, B // 2 + np.arange(0, n - B + 1, 37), n - (B - B // 2 - 1):n]
    sub = np.unique(pick)
    # the oracle on every 37th node of the large request and on all the others
    req = np.searchsorted(case.node_off, sub, side="right") - 1
    case.h, case.depth = case.h[sub], case.depth[sub]
    case.node_off = np.searchsorted(req, np.arange(B + 1)).astype(np.int32)
    compare(case, {k: v[sub] for k, v in got[0].items()}, run_oracle(case), H_TOL[dtype],
            label=f"uneven {dtype} B={B} M={M} d_m={d_m}")


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_loose_node_bound_of_a_large_batch(lib, dtype):
    """16384 requests of 4 nodes under t_max = 65536: the grid follows the nodes there are (with
    a block per chunk that the bound allows it would be past what a launch may hold)."""
    B, T, d, d_m = 16384, 4, 64, 64
    wl = _wl(dtype, B=1, T=1, M=8, d=d, d_m=d_m, d_c=64, k_max=4)
    W = make_case(wl, affine="unit").weights
    fv = lib.Fovea(dims_of(wl, W, 1 if dtype == "bf16" else 0), W, device="cuda")
    g = torch.Generator(device="cuda").manual_seed(5)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda").to(dt)  # noqa: E731
    ar = torch.arange(B + 1, device="cuda")
    inp = dict(mem_off=ar * 8, keys=rnd(B * 8, d_m), values=rnd(B * 8, d_m), valid=None,
               node_off=(ar * T).to(torch.int32), h=rnd(B * T, d),
               depth=torch.zeros(B * T, dtype=torch.int32, device="cuda"), tau=torch.full((B,), 0.7, device="cuda"),
               m_max=8, k_min=1, k_max=4)
    got = []
    for t_max in (T, B * T):
        print(f"[gpu] loose bound {dtype} B={B} t_max={t_max}", flush=True)
        out = fv.retrieve_fuse(dict(inp, t_max=t_max))
        torch.cuda.synchronize()
        got.append(gpu_outputs(out))
        assert lib.fovea_last_error(fv.ctx)[0] == 0
    fv.close()
    for k in got[0]:
        assert np.array_equal(got[0][k], got[1][k]), k
