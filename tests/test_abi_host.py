"""CPU-side checks of the product library: it loads, exports every declared symbol, rejects bad
arguments before touching a GPU, and its host arithmetic (Adam, bf16 rounding, rotary tables)
matches the oracle.  No GPU compute is launched here."""
import ctypes
import math
import os
import re
import time

import numpy as np
import pytest

import paper_2604_05091_amd as mt
from paper_2604_05091_amd.binding import ModelCfg

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_symbols():
    names = set()
    for hdr in ("megatrain.h", "megatrain_kernels.h"):
        text = open(os.path.join(ROOT, "include", hdr)).read()
        text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
        names |= set(re.findall(r"\b(mt_[a-z0-9_]+)\s*\(", text))
    return sorted(names)


def test_library_exports_every_declared_symbol():
    L = ctypes.CDLL(mt.lib_path())
    syms = declared_symbols()
    assert len(syms) >= 30
    for s in syms:
        assert hasattr(L, s), f"{s} is declared in include/ but not exported"


def test_tensor_table_matches_the_input_module():
    import mt_inputs
    L = mt.lib()
    for name in ("tiny", "14B"):
        shape, B, T = mt_inputs.CONFIGS[name]
        cfg = ModelCfg.make(shape.n_layers, shape.hidden, shape.n_q_heads, shape.n_kv_heads, shape.head_dim, shape.ffn,
                            shape.vocab, B, T)
        n = ctypes.c_int32()
        assert L.mt_tensor_count(ctypes.byref(cfg), ctypes.byref(n)) == 0
        table = mt_inputs.tensor_table(shape)
        assert n.value == len(table) == 9 * shape.n_layers + 3
        for i, (nm, r, c) in enumerate(table):
            rr, cc, p = ctypes.c_int64(), ctypes.c_int64(), ctypes.c_char_p()
            assert L.mt_tensor_info(ctypes.byref(cfg), i, ctypes.byref(rr), ctypes.byref(cc), ctypes.byref(p)) == 0
            assert (p.value.decode(), rr.value, cc.value) == (nm, r, c)
        assert L.mt_tensor_info(ctypes.byref(cfg), n.value, ctypes.byref(rr), ctypes.byref(cc), None) == -1


def test_create_rejects_bad_configurations_without_a_gpu():
    L = mt.lib()
    h = ctypes.c_void_p()
    good = dict(n_layers=2, hidden=256, n_q_heads=4, n_kv_heads=4, head_dim=64, ffn=688, vocab=1024, max_batch=2,
                max_seq=128)
    dummy = (ctypes.c_void_p * 21)(*([1] * 21))

    def create(**kw):
        cfg = ModelCfg.make(**{**good, **kw})
        return L.mt_create(ctypes.byref(cfg), dummy, ctypes.byref(h))

    assert L.mt_create(None, dummy, ctypes.byref(h)) == -1
    assert create(n_layers=0) == -1
    assert create(n_q_heads=4, n_kv_heads=3) == -1
    assert create(head_dim=96) == -2
    assert create(ffn=690) == -2
    assert create(ckpt_interval=0) == -1
    assert create(max_seq=100) == -2
    assert create(rms_eps=0.0) == -1
    cfg = ModelCfg.make(**good)
    cfg.struct_size = 8
    assert L.mt_create(ctypes.byref(cfg), dummy, ctypes.byref(h)) == -1
    cfg = ModelCfg.make(**good)
    assert L.mt_create(ctypes.byref(cfg), None, ctypes.byref(h)) == -1
    assert b"host_param_ptrs" in L.mt_last_error()
    # the arena plan is checked against the cap before any device call
    assert create(max_device_bytes=1 << 20) == -4
    assert b"device arena" in L.mt_last_error()
    assert L.mt_destroy(None) == 0
    assert L.mt_adam_step(None, 1e-3, 0.9, 0.999, 1e-8, 0.0, 1) == -1
    assert L.mt_train_step(None, None, None, 1, 8, None) == -1


def test_host_adam_matches_oracle(orc64):
    L = mt.lib()
    rng = np.random.default_rng(0)
    n = 200_003                                  # several thread chunks and a ragged tail
    p0 = (rng.standard_normal(n) * 0.02).astype(np.float32)
    p, m, v = p0.copy(), np.zeros(n, np.float32), np.zeros(n, np.float32)
    pr, mr, vr = p0.astype(np.float64), np.zeros(n), np.zeros(n)
    shadow = np.zeros(n, np.uint16)
    for t, wd in ((1, 0.0), (2, 0.01), (3, 0.01)):
        g = (rng.standard_normal(n) * 1e-3).astype(np.float32)
        assert L.mt_k_host_adam(p.ctypes.data, g.ctypes.data, m.ctypes.data, v.ctypes.data, shadow.ctypes.data, n,
                                1e-4, 0.9, 0.999, 1e-8, wd, t) == 0
        # the C ABI takes float arguments: give the oracle the same (float-rounded) hyper-parameters
        f = lambda x: float(np.float32(x))
        orc64.adam(pr, g.astype(np.float64), mr, vr, f(1e-4), f(0.9), f(0.999), f(1e-8), f(wd), t)
    assert np.linalg.norm(p - pr) / np.linalg.norm(pr) < 1e-6
    upd, upd_ref = p.astype(np.float64) - p0, pr - p0
    assert np.linalg.norm(upd - upd_ref) / np.linalg.norm(upd_ref) < 1e-4     # the update itself, not just p
    assert np.linalg.norm(m - mr) / np.linalg.norm(mr) < 1e-6 and np.linalg.norm(v - vr) / np.linalg.norm(vr) < 1e-6
    # the bf16 copy is the updated parameter rounded to nearest even
    import torch
    ref_bits = torch.from_numpy(p).to(torch.bfloat16).view(torch.int16).numpy().view(np.uint16)
    assert np.array_equal(shadow, ref_bits)
    assert L.mt_k_host_adam(p.ctypes.data, g.ctypes.data, m.ctypes.data, v.ctypes.data, None, n, 1e-4, 0.9, 0.999,
                            1e-8, 0.0, 0) == -1


def test_host_adam_from_two_threads_at_once_equals_one_at_a_time():
    """The host pool runs one job at a time; a caller that finds it busy (the optimizer thread next to the weight
    packing thread) spawns threads of its own.  Both take chunks from a shared counter.  Two updates issued at the
    same moment must give, bit for bit, what the same updates give one after the other."""
    import threading
    L = mt.lib()
    rng = np.random.default_rng(5)
    n = 3_000_017                                # ~46 chunks of 65536 with a ragged tail
    def fresh(seed):
        r = np.random.default_rng(seed)
        return [(r.standard_normal(n) * 0.02).astype(np.float32), (r.standard_normal(n) * 1e-3).astype(np.float32),
                np.zeros(n, np.float32), np.zeros(n, np.float32), np.zeros(n, np.uint16)]
    def run(a, reps):
        for t in range(1, reps + 1):
            assert L.mt_k_host_adam(a[0].ctypes.data, a[1].ctypes.data, a[2].ctypes.data, a[3].ctypes.data,
                                    a[4].ctypes.data, n, 1e-3, 0.9, 0.999, 1e-8, 0.01, t) == 0
    ref = [fresh(1), fresh(2)]
    for a in ref:
        run(a, 3)
    got = [fresh(1), fresh(2)]
    th = [threading.Thread(target=run, args=(a, 3)) for a in got]
    for t in th:
        t.start()
    for t in th:
        t.join()
    for a, b in zip(ref, got):
        for x, y in zip(a, b):
            assert np.array_equal(x, y)
    assert not np.array_equal(got[0][0], fresh(1)[0])


def test_host_bf16_rounding_is_nearest_even():
    import torch
    L = mt.lib()
    rng = np.random.default_rng(1)
    x = np.concatenate([rng.standard_normal(100_000).astype(np.float32) * 10,
                        np.array([0.0, -0.0, 1.0, 1.00390625, 1.01171875, 3.4e38, 1e-40, np.inf, -np.inf], np.float32)])
    out = np.zeros(x.size, np.uint16)
    assert L.mt_k_host_f32_to_bf16(out.ctypes.data, x.ctypes.data, x.size) == 0
    ref = torch.from_numpy(x).to(torch.bfloat16).view(torch.int16).numpy().view(np.uint16)
    assert np.array_equal(out, ref)


@pytest.mark.parametrize("hd,base", [(64, 10000.0), (128, 1.0e6)])
def test_rope_table_matches_oracle_rotation(orc64, hd, base):
    """cos/sin at (t, j) must be what the oracle's rotation does to the unit vector of pair j."""
    L = mt.lib()
    T = 4096
    cs, sn = np.empty((T, hd // 2), np.float32), np.empty((T, hd // 2), np.float32)
    assert L.mt_k_rope_table(cs.ctypes.data, sn.ctypes.data, T, hd, base) == 0
    x = np.zeros((T, hd))
    x[:, : hd // 2] = 1.0
    y = orc64.rope(x, 1, T, 1, hd, base, +1)
    assert np.max(np.abs(y[:, : hd // 2] - cs)) < 6e-8 and np.max(np.abs(y[:, hd // 2:] - sn)) < 6e-8
    assert L.mt_k_rope_table(cs.ctypes.data, sn.ctypes.data, T, 63, base) == -1


def test_model_flops_formula_reproduces_the_paper_rows():
    rows = [l.split() for l in open(os.path.join(ROOT, "tests", "golden", "paper_table7_flops.txt"))
            if l.strip() and not l.startswith("#")]
    for ctx, bs, secs, tflops in rows:
        f = mt.model_flops(n_params=7.62e9, n_layers=28, hidden=3584, batch=int(bs), seq=int(ctx))
        assert abs(f / float(secs) / 1e12 / float(tflops) - 1) < 0.015, (ctx, f / float(secs) / 1e12, tflops)


def test_reductions_are_shared_in_the_measured_range_only():
    """Up to 8192 rows and columns, and wider results in one round of tiles; where the estimate is well below that of the other kernels."""
    sharers = lambda form, M, N, K: mt.binding.lib().mt_k_gemm_sharers(form, M, N, K, N)
    assert sharers(0, 8192, 64, 2048) > 1 and sharers(0, 32, 8192, 4096) > 1 and sharers(0, 32, 12288, 4096) > 1 and sharers(1, 600, 600, 4104) > 1
    for form, M, N, K in ((0, 8193, 64, 2048), (0, 41236, 8, 7664), (1, 35575, 8, 7048), (0, 12887, 24, 8648), (0, 49152, 64, 8192),
                          (0, 1248, 648, 712), (0, 3896, 192, 784), (0, 48, 15712, 2816), (0, 120, 9000, 2048),   # (too little to gain, or to lose with operands in the caches)
                          (0, 32, 16448, 4096), (0, 29, 16848, 4608), (0, 20, 17584, 24640), (1, 600, 600, 4096)):
        assert sharers(form, M, N, K) == 1, (form, M, N, K)


def test_attention_queries_agree():
    """mt_k_flash_route, mt_k_flash_sets and mt_k_flash_lists speak of the same kernels, those that run: (1, 1032, 4, 1, 128) takes blocks of 32 rows."""
    L = mt.binding.lib()
    seen = set()
    for hd in (64, 128):
        for T in (8, 64, 72, 136, 264, 520, 1032, 2056):
            for B in (1, 3, 13, 40, 100):
                for Hq, Hkv in ((2, 2), (4, 1), (9, 3), (16, 16)):
                    r, sets, lists = (ctypes.c_int32 * 3)(), (ctypes.c_int32 * 6)(), (ctypes.c_int32 * 3)()
                    for query, out in ((L.mt_k_flash_route, r), (L.mt_k_flash_sets, sets), (L.mt_k_flash_lists, lists)):
                        assert query(B, T, Hq, Hkv, hd, ctypes.addressof(out)) == 0
                    assert tuple(r) == tuple(sets[::2])
                    for i in range(3):
                        assert not lists[i] or sets[2 * i:2 * i + 2] == [256, 1]
                        seen.add((hd, i, sets[2 * i], sets[2 * i + 1], lists[i]))
    for hd, n in ((64, 8), (128, 4)):
        for i in range(3):
            assert {(hd, i, 256, 1, 0), (hd, i, 256, 1, 1), (hd, i, 128, 2, 0), (hd, i, 64, 4, 0), (hd, i, 32, n, 0)} <= seen
    r = (ctypes.c_int32 * 3)()
    assert L.mt_k_flash_route(1, 1032, 4, 1, 128, ctypes.addressof(r)) == 0 and list(r) == [32, 32, 32]
    assert L.mt_k_flash_lists(1, 1032, 3, 2, 128, ctypes.addressof(r)) != 0
    assert L.mt_k_flash_together(1, 520, 8, 2, 64) == 1 and L.mt_k_flash_together(16, 4096, 32, 32, 128) == 0 and L.mt_k_flash_together(1, 520, 3, 2, 64) < 0


def _dealt_group(n_sets, copies, n_blocks, tiles):
    """The grouping of the attention's lists of blocks, weighed slot by slot: the blocks of an XCD are dealt to 32 workers back and forth."""
    per_set, p = copies * n_blocks, 1
    while p < 8 and -(-n_sets * p // 8) * 8 * 100 > n_sets * p * 107:
        p *= 2
    n_parts, per_part = -(-n_sets * p // 8), -(-per_set // p)
    workers = min(32, n_parts * per_part)
    group, best, best_t = 1, 1, None
    while True:
        sums, w, step = [0] * workers, 0, 1
        for g0 in range(0, n_parts, group):
            for i in range(per_part):
                t = 1 + tiles(min(per_set - 1, i * p) // copies)
                for _ in range(min(group, n_parts - g0)):
                    sums[w] += t
                    w += step
                    if w == workers or w < 0:
                        w, step = w - step, -step
        t = max(sums) * (1 + 0.004 * min(group, 32))
        if best_t is None or t < best_t:
            best, best_t = group, t
        if group == n_parts:
            return best
        group = min(2 * group, n_parts)


def test_lists_of_attention_blocks_are_grouped_as_weighed_slot_by_slot():
    L, rng, n, groups = mt.binding.lib(), np.random.default_rng(5), 0, set()
    for _ in range(400):
        B, T, Hkv, G = int(2 ** rng.uniform(0, 8)), 8 * int(2 ** rng.uniform(3, 9)), int(rng.integers(1, 33)), int(rng.choice([1, 2, 3, 4, 8]))
        if B * Hkv * G * -(-T // 256) > 20000:
            continue
        lists = (ctypes.c_int32 * 3)()
        assert L.mt_k_flash_lists(B, T, Hkv * G, Hkv, 128, ctypes.addressof(lists)) == 0
        nb, nt = -(-T // 256), -(-T // 64)
        want = (_dealt_group(B * Hkv, G, nb, lambda r: min(nt, 4 * (nb - r))) if lists[0] or lists[1] else 0,
                _dealt_group(B * Hkv, 1, nb, lambda r: G * (nt - 4 * r)) if lists[2] else 0)
        for got, w in zip(lists, (want[0], want[0], want[1])):
            assert got in (0, w), (B, T, Hkv, G)
        n += sum(map(bool, lists))
        groups |= set(lists)
    assert n > 200 and len(groups) > 6


def test_lists_of_attention_blocks_take_the_caller_no_time():
    """Three lists of up to 65 000 blocks an XCD are grouped in less than a tenth of the 2.5 ms that weighing them slot by slot took."""
    L, lists, best = mt.binding.lib(), (ctypes.c_int32 * 3)(), 1.0
    for _ in range(20):
        t = time.perf_counter()
        assert L.mt_k_flash_lists(16000, 72, 32, 32, 128, ctypes.addressof(lists)) == 0
        best = min(best, time.perf_counter() - t)
    assert all(lists) and best < 250e-6, best
