"""GPU parity of kv_decode_attention (attention of a generated token over the compacted cache)
against the oracle, on seeded synthetic caches and on the cache the eviction pass compacts.

Tolerance: the kernel forms logits, the softmax and the weighted sum in fp32.  A logit of a d = 128
dot product carries an error of a few fp32 ulps of sum |q_i k_i| (about 1e-6 here), which moves each
softmax weight by about that fraction; the output, a convex combination of value rows, moves by at
most that times max |v|.  The test allows 2e-5 max|v| + 1e-5 |o|.
"""
import numpy as np
import pytest

from oracle import decode, evict
from paper_2609_30738_amd import _lib, api, workloads
from tests import gpu_cases

pytestmark = pytest.mark.gpu


def _dev(x):
    return api.to_device(np.ascontiguousarray(x))


def _check_out(out, di, k_host, v_host, lens, append, where):
    """Compare every (problem, head) output with the oracle over the rows in use."""
    o = out.reshape(len(lens), di.h_q, di.d)
    for p, L in enumerate(lens):
        kd = evict.decode(k_host[p, :, :L], di.dtype)
        vd = evict.decode(v_host[p, :, :L], di.dtype)
        qd = evict.decode(di.q[p], di.dtype)
        kn = evict.decode(di.k_new[p], di.dtype) if append else None
        vn = evict.decode(di.v_new[p], di.dtype) if append else None
        ref = decode.decode_attention(qd, kd, vd, di.scale, kn, vn)
        vmax = max(np.abs(vd).max() if L else 0.0, np.abs(vn).max() if append else 0.0)
        err = np.abs(o[p] - ref)
        bound = 2e-5 * vmax + 1e-5 * np.abs(ref)
        assert np.all(err <= bound), (f"{where} p={p} L={L}: worst error {err.max():.3g} at "
                                      f"{np.unravel_index(np.argmax(err - bound), err.shape)}")


def _run(di, append=True, where=""):
    import torch
    print(f"[gpu case] decode {where} dtype={di.dtype} h_q={di.h_q} h_kv={di.h_kv} d={di.d} "
          f"stride={di.row_stride} lens={list(di.lens)} append={append}", flush=True)
    cb = _lib.CacheBatch(di.dtype, di.h_q, di.h_kv, di.d, di.row_stride, di.lens)
    k, v = _dev(di.k), _dev(di.v)
    out = torch.empty(len(di.lens) * di.h_q * di.d, dtype=torch.float32, device="cuda")
    ws = torch.empty(max(_lib.decode_workspace_bytes(cb), 256), dtype=torch.uint8, device="cuda")
    _lib.decode_attention(cb, _dev(di.q), k, v, _dev(di.k_new) if append else None,
                          _dev(di.v_new) if append else None, di.scale, out, ws)
    torch.cuda.synchronize()
    return out.cpu().numpy(), api.to_host_bits(k), api.to_host_bits(v)


@pytest.mark.parametrize("dtype,d,h_q,h_kv", [("bf16", 128, 32, 8), ("bf16", 64, 8, 4),
                                              ("f32", 128, 4, 4), ("f32", 64, 16, 2),
                                              ("bf16", 128, 12, 4)])
@pytest.mark.parametrize("append", [True, False])
def test_decode_matches_oracle(dtype, d, h_q, h_kv, append):
    """Group sizes 1, 2, 3 (padded to 4), 4 and 8; lengths 1 .. 300 in one batch, including rows
    that leave a partial pass and a partial unrolled block."""
    lens = [1, 7, 96, 300, 130, 65]
    di = workloads.draw_decode(dtype, h_q, h_kv, d, 320, lens, seed=3)
    out, k_after, v_after = _run(di, append, "shapes")
    _check_out(out, di, di.k, di.v, lens, append, f"{dtype} d={d} G={h_q // h_kv}")
    if append:
        for p, L in enumerate(lens):  # row L now holds the new token; nothing else changed
            np.testing.assert_array_equal(k_after[p, :, L], di.k_new[p])
            np.testing.assert_array_equal(v_after[p, :, L], di.v_new[p])
            np.testing.assert_array_equal(np.delete(k_after[p], L, axis=1), np.delete(di.k[p], L, axis=1))
            np.testing.assert_array_equal(np.delete(v_after[p], L, axis=1), np.delete(di.v[p], L, axis=1))
    else:
        np.testing.assert_array_equal(k_after, di.k)
        np.testing.assert_array_equal(v_after, di.v)


def test_decode_generation_steps_append_in_place():
    """Four generated tokens in a row over the same cache buffers: each call appends its row and
    the next call attends to it from the cache."""
    import torch
    lens = [96, 40, 250]
    first = workloads.draw_decode("bf16", 32, 8, 128, 260, lens, seed=10)
    cb = _lib.CacheBatch("bf16", 32, 8, 128, 260, lens)
    k, v = _dev(first.k), _dev(first.v)
    k_ref, v_ref = first.k.copy(), first.v.copy()
    out = torch.empty(len(lens) * 32 * 128, dtype=torch.float32, device="cuda")
    ws = torch.empty(max(_lib.decode_workspace_bytes(cb), 256), dtype=torch.uint8, device="cuda")
    for step in range(4):
        di = workloads.draw_decode("bf16", 32, 8, 128, 260, lens, seed=100 + step)
        cur = [int(x) for x in cb.lens_host]
        print(f"[gpu case] decode step {step} lens={cur}", flush=True)
        _lib.decode_attention(cb, _dev(di.q), k, v, _dev(di.k_new), _dev(di.v_new), di.scale, out,
                              ws)
        torch.cuda.synchronize()
        _check_out(out.cpu().numpy(), di, k_ref, v_ref, cur, True, f"step {step}")
        for p, L in enumerate(cur):
            k_ref[p, :, L] = di.k_new[p]
            v_ref[p, :, L] = di.v_new[p]
        cb.advance()
    np.testing.assert_array_equal(api.to_host_bits(k), k_ref)
    np.testing.assert_array_equal(api.to_host_bits(v), v_ref)


def test_decode_long_cache_splits_rows():
    """An uncompacted 20000-row cache next to a 777-row one (few units: the rows are split over
    workgroups and the partials merged)."""
    lens = [20000, 777]
    di = workloads.draw_decode("bf16", 32, 8, 128, 20001, lens, seed=5)
    cb = _lib.CacheBatch("bf16", 32, 8, 128, 20001, lens)
    assert _lib.decode_workspace_bytes(cb) > 0
    out, _, _ = _run(di, True, "long")
    _check_out(out, di, di.k, di.v, lens, True, "long")


@pytest.mark.parametrize("dtype,d,h_q,h_kv", [("bf16", 128, 8, 2), ("bf16", 64, 4, 4),
                                              ("bf16", 128, 16, 2), ("f32", 128, 4, 2),
                                              ("f32", 64, 8, 1)])
def test_decode_splits_with_rising_logits(dtype, d, h_q, h_kv):
    """Caches of 1 .. 1500 rows cut into splits of 128 and 192 rows (empty splits, a split of one
    row, whole and partial steps, the appended row alone in its split), with logits that rise from
    -16 to 16 nats along the rows of every second problem, so that the reference of the weights is
    raised many times.  A logit of 16 nats from terms of like sign errs by at most
    (d + 2) 2^-24 16 < 1.3e-4 in the worst order and a few 2^-24 16 = 4e-6 in a blocked one, inside
    the module's 2e-5 max|v|."""
    lens = [1500, 128, 127, 1, 383, 1344]
    di = workloads.draw_decode(dtype, h_q, h_kv, d, 1502, lens, seed=21)
    G = h_q // h_kv
    q = evict.decode(di.q, dtype)
    for p in range(0, len(lens), 2):
        for g in range(h_kv):
            u = q[p, g * G]
            ramp = np.linspace(-16.0, 16.0, lens[p])[:, None] / (di.scale * float(u @ u))
            rows = (ramp * u[None]).astype(np.float32)
            di.k[p, g, :lens[p]] = workloads.f32_to_bf16_bits(rows) if dtype == "bf16" else rows
    for append in (True, False):
        out, k_after, _ = _run(di, append, "splits")
        _check_out(out, di, di.k, di.v, lens, append, f"splits {dtype} d={d} G={G}")
        if append:
            for p, L in enumerate(lens):
                np.testing.assert_array_equal(k_after[p, :, L], di.k_new[p])


def test_decode_over_the_compacted_cache_of_the_pass():
    """Eviction pass on the GPU (one Mistral layer, L = 3000, B = 64), compaction into blocks with
    room for generated rows, then one decode step; compared with the oracle's compacted rows and
    decode attention for every kv head whose admissions equal the oracle's."""
    import torch
    wl = workloads.mistral_layer()
    wl.seq_lens = [3000]
    pk = workloads.draw_packed(wl)
    lam1, lam2 = gpu_cases.layer_lambdas(wl, [0])
    inp = api.upload(wl.dtype, wl.h_q, wl.h_kv, wl.d, wl.w, pk.q_win, pk.k, pk.v, pk.lens,
                     pk.tok_off, lam1, lam2)
    out = api.allocate(inp, wl.budget)
    print("[gpu case] decode after the eviction pass L=3000", flush=True)
    api.run_pass(inp, out, wl.budget)
    stride = wl.budget + wl.w + 2
    kc = torch.empty(wl.h_kv * stride * wl.d, dtype=inp.k.dtype, device="cuda")
    vc = torch.empty_like(kc)
    _lib.compact_cache_ex(inp.batch, inp.k, inp.v, out.sel_idx, wl.budget, wl.w, None, kc, vc,
                          out_rows=stride)
    di = workloads.draw_decode("bf16", wl.h_q, wl.h_kv, wl.d, stride, [wl.budget + wl.w], seed=9)
    cb = _lib.CacheBatch("bf16", wl.h_q, wl.h_kv, wl.d, stride, [wl.budget + wl.w])
    o = torch.empty(wl.h_q * wl.d, dtype=torch.float32, device="cuda")
    _lib.decode_attention(cb, _dev(di.q), kc, vc, _dev(di.k_new), _dev(di.v_new), di.scale, o)
    torch.cuda.synchronize()
    sel = out.sel_idx.cpu().numpy().reshape(wl.h_kv, wl.budget)
    L = 3000
    k = pk.k.reshape(wl.h_kv, L, wl.d)
    v = pk.v.reshape(wl.h_kv, L, wl.d)
    res = evict.evict_problem(pk.q_win[0], k, v, wl.dtype, wl.scale, float(lam1[0]),
                              float(lam2[0]), wl.budget)
    o = o.cpu().numpy().reshape(wl.h_q, wl.d)
    G = wl.h_q // wl.h_kv
    same = 0
    for g in range(wl.h_kv):
        if set(sel[g].tolist()) != set(res.heads[g].trace.selected):
            continue  # a near-tie admitted another row: its cache differs legitimately
        same += 1
        kd = evict.decode(res.k_out[g][None], wl.dtype)
        vd = evict.decode(res.v_out[g][None], wl.dtype)
        ref = decode.decode_attention(evict.decode(di.q[0, g * G:(g + 1) * G], wl.dtype), kd, vd,
                                      di.scale, evict.decode(di.k_new[0, g:g + 1], wl.dtype),
                                      evict.decode(di.v_new[0, g:g + 1], wl.dtype))
        vmax = max(np.abs(vd).max(), np.abs(evict.decode(di.v_new[0, g], wl.dtype)).max())
        err = np.abs(o[g * G:(g + 1) * G] - ref)
        assert np.all(err <= 2e-5 * vmax + 1e-5 * np.abs(ref)), f"g={g}: {err.max():.3g}"
    assert same >= wl.h_kv - 1, f"only {same} kv heads admitted the oracle's rows"


@pytest.mark.parametrize("dtype,d,h_q", [("bf16", 128, 32), ("bf16", 64, 8), ("f32", 128, 8), ("f32", 64, 64)])
def test_decode_of_values_near_the_largest_float(dtype, d, h_q):
    """Values of 2^118 in every row and logits 7 octaves higher from row 200 on: the weighted sums stay
    finite because no weight exceeds 1 (301 rows of 2^118 sum to less than 2^127), and the output is 2^118."""
    lens = [300, 260]
    di = workloads.draw_decode(dtype, h_q, 8, d, 301, lens, seed=4)
    q = evict.decode(di.q, dtype)
    u = q[:, ::h_q // 8]  # one head of each group
    rows = np.zeros(di.k.shape, dtype=np.float32)
    rows[:, :, 200:] = (7 * np.log(2) / (di.scale * np.sum(u * u, -1, keepdims=True)) * u)[:, :, None]
    v = np.full(di.v.shape, 2.0 ** 118, dtype=np.float32)
    bits = workloads.f32_to_bf16_bits if dtype == "bf16" else np.asarray
    di.k[:], di.v[:] = bits(rows), bits(v)
    for append in (False, True):
        if append:
            di.v_new[:] = bits(np.full(di.v_new.shape, 2.0 ** 118, dtype=np.float32))
        out, _, _ = _run(di, append, "large values")
        np.testing.assert_allclose(out, 2.0 ** 118, rtol=1e-5)


@pytest.mark.parametrize("dtype,d,h_q,n_prob,rows,splits", [
    ("bf16", 128, 32, 32, 9300, 9), ("bf16", 64, 8, 32, 9300, 9), ("f32", 64, 16, 32, 9300, 9),
    ("f32", 128, 8, 32, 9300, 9), ("bf16", 128, 64, 4, 33000, 24)])
@pytest.mark.parametrize("append", [False, True])
def test_decode_over_caches_larger_than_the_chip(dtype, d, h_q, n_prob, rows, splits, append):
    """K and V of 256 MiB and more (read past the caches), unequal lengths, in about three rounds of
    splits (256 units of at least 1024 rows a split) and in one: the longest, the shortest and a few
    other problems against the oracle."""
    import torch
    h_kv, stride = 8, rows + 1
    assert 2 * n_prob * h_kv * rows * d * (2 if dtype == "bf16" else 4) >= 256 << 20
    lens = [rows - 97 * p if p % 5 else rows - 31 * p for p in range(n_prob - 1)] + [1]
    print(f"[gpu case] decode past the caches dtype={dtype} h_q={h_q} d={d} lens={lens[:3]}.. "
          f"x{n_prob} append={append}", flush=True)
    cb = _lib.CacheBatch(dtype, h_q, h_kv, d, stride, lens)
    need = n_prob * h_q * splits * (d + 2) * 4
    assert _lib.decode_workspace_bytes(cb) == -(-need // 256) * 256
    gen = torch.Generator(device="cuda")
    gen.manual_seed(11)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=gen).to(dt)
    q, k, v = rnd(n_prob, h_q, d), rnd(n_prob, h_kv, stride, d), rnd(n_prob, h_kv, stride, d)
    k[:, :, ::1000] *= 4  # a few dominant rows
    kn, vn = (rnd(n_prob, h_kv, d), rnd(n_prob, h_kv, d)) if append else (None, None)
    out = torch.empty(n_prob * h_q * d, dtype=torch.float32, device="cuda")
    ws = torch.empty(_lib.decode_workspace_bytes(cb), dtype=torch.uint8, device="cuda")
    k0, v0 = k.clone(), v.clone()
    _lib.decode_attention(cb, q, k, v, kn, vn, d ** -0.5, out, ws)
    torch.cuda.synchronize()
    o = out.cpu().numpy().reshape(n_prob, h_q, d)
    host = lambda x: x.float().cpu().numpy().astype(np.float64)
    for p in (0, 1, n_prob // 2, n_prob - 1):
        L = lens[p]
        kd, vd = host(k0[p, :, :L]), host(v0[p, :, :L])
        ref = decode.decode_attention(host(q[p]), kd, vd, d ** -0.5, host(kn[p]) if append else None,
                                      host(vn[p]) if append else None)
        vmax = max(np.abs(vd).max(), np.abs(host(vn[p])).max() if append else 0.0)
        err = np.abs(o[p] - ref)
        assert np.all(err <= 2e-5 * vmax + 1e-5 * np.abs(ref)), f"p={p} L={L}: worst error {err.max():.3g}"
    if append:  # row L of every block is the new token's, nothing else changed
        at = torch.tensor(lens, device="cuda")
        i = torch.arange(n_prob, device="cuda")
        k0[i, :, at], v0[i, :, at] = kn, vn
    assert torch.equal(k, k0) and torch.equal(v, v0)
