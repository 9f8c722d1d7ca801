"""The rules that choose a kernel variant by size (csrc/fd_rules.h), compiled for the CPU: each
rule on both sides of its lines, at sizes where both variants were measured on an MI355X.  The
attention's schedule (csrc/fd_attn_sched.h) runs every tile-step exactly once, whole or cut."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2607_12121_amd", "csrc")
CUS = 256

SHIM = r"""
#include "fd_attn_sched.h"
#include "fd_gemm_rules.h"
namespace {
// Every piece of every share as attn_fwd_kernel walks them, eight numbers each: share, head, query
// tile, request, first and last + 1 key tile, scratch slot, and for a first piece, from which the
// merge starts, the item's last share.
template <int QB, int DH, bool TABLES, bool CUT>
int pieces(const int32_t* cu_q, const int32_t* tok, int B, int H, int G, int nkv_max, int* out, int cap, int* cut) {
  static fd::SchedTables t;
  t.tpre[0] = 0;
  t.wpre[0] = 0;
  for (int b = 0; b < B; ++b) {
    const int nt = (cu_q[b + 1] - cu_q[b] + QB - 1) / QB;
    t.tpre[b + 1] = t.tpre[b] + nt;
    t.wpre[b + 1] = t.wpre[b] + static_cast<long long>(nt) * ((tok[b + 1] - tok[b] + 63) / 64);
  }
  const fd::AttnSched<QB, DH, TABLES, CUT> s(&t, cu_q, tok, B, H, G, nkv_max);
  *cut = s.cut;
  int n = 0;
  if (s.tiles == 0) return 0;
  for (int blk = 0; blk < G; ++blk) {
    const int w = s.share(blk);
    long long p = s.bound(w);
    const long long p_end = s.bound(w + 1);
    while (p < p_end) {
      long long i0;
      int nkv, head, b, first, tau;
      s.locate(p, i0, nkv, head, b, first, tau);
      const long long i1 = i0 + nkv, e = p_end < i1 ? p_end : i1;
      if (n == cap) return -1;
      const int k0 = static_cast<int>(p - i0), k1 = static_cast<int>(e - i0);
      const int row[8] = {w, head, tau, b, k0, k1, s.slot_of(w, k0, k1, nkv), k0 == 0 && k1 < nkv ? s.last_share(w, i1) : -1};
      for (int k = 0; k < 8; ++k) out[8 * n + k] = row[k];
      ++n;
      p = e;
    }
  }
  return n;
}
}  // namespace
extern "C" {
int score_one_pass(int regions, long long values, int cus) { return fd::score_one_pass(regions, values, cus); }
int attn_cuts(int dh, int tiles, int heads, long long work_head, int nkv_max, int G) {
  return fd::attn_cuts(dh, tiles * heads, heads, work_head, tiles, (work_head * heads + G - 1) / G, nkv_max, G, 0);
}
int gemm_large(int n_max, int N) { return fd::gemm_large(n_max, N, false); }
int large_shape(int M, int N, int K, int cus) { return fd::large_shape(M, N, K, cus, 4 * cus); }
int small_shape(int M, int N, int K, int cus) { return fd::small_shape(M, N, K, 2 * cus, 4 * cus); }
// K splits of one product
int gemm_splits(int n_max, int M, int N, int K, int cus) {
  const bool large = fd::gemm_large(n_max, N, false);
  if (!fd::gemm_may_split(n_max, N, large)) return 1;
  return fd::choose_split(((M + 127) / 128) * ((N + 127) / 128), K / fd::TBK, large ? cus : 2 * cus, 4 * cus);
}
int attn_may_cut(int dh, int heads, int requests, long long tokens, int max_request_tokens, int G) {
  return fd::attn_may_cut(dh, heads, requests, tokens, max_request_tokens, 256, G);
}
int attn_slot_at(int x, int j) { return fd::AttnSched<256, 64, true, true>::slot_at(x, j); }
long long div_steps(long long q, long long d) { return fd::div_steps(q, d); }
int attn_pieces(int dh, int tables, int may_cut, const int32_t* cu_q, const int32_t* tok, int B, int H, int G, int nkv_max,
                int* out, int cap, int* cut) {
#define RUN(QB, DH)                                                                                                      \
  (tables ? (may_cut ? pieces<QB, DH, true, true>(cu_q, tok, B, H, G, nkv_max, out, cap, cut)                            \
                     : pieces<QB, DH, true, false>(cu_q, tok, B, H, G, nkv_max, out, cap, cut))                          \
          : (may_cut ? pieces<QB, DH, false, true>(cu_q, tok, B, H, G, nkv_max, out, cap, cut)                           \
                     : pieces<QB, DH, false, false>(cu_q, tok, B, H, G, nkv_max, out, cap, cut)))
  return dh == 16 ? RUN(128, 16) : dh == 64 ? RUN(256, 64) : RUN(256, 128);
#undef RUN
}
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("needs a C++ compiler")
    d = tmp_path_factory.mktemp("rules")
    src, so = d / "rules.cpp", d / "rules.so"
    src.write_text(SHIM)
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", f"-I{CSRC}", str(src), "-o", str(so)],
                   check=True)
    lib = ctypes.CDLL(str(so))
    lib.score_one_pass.argtypes = [ctypes.c_int, ctypes.c_longlong, ctypes.c_int]
    lib.div_steps.argtypes = [ctypes.c_longlong] * 2
    lib.div_steps.restype = ctypes.c_longlong
    lib.attn_may_cut.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_longlong, ctypes.c_int, ctypes.c_int]
    lib.attn_cuts.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_longlong, ctypes.c_int, ctypes.c_int]
    return lib


@pytest.mark.parametrize("regions,values,one_pass", [
    (1, 8192, True), (64, 8192, True), (511, 8192, True),
    # few large regions are cut: one pass took up to 2.3 times as long
    (1, 65536, False), (4, 65536, False), (16, 16 * 1024, False), (16, 65536, False), (64, 16384, False), (64, 65536, False),
    (127, 16384, False), (140, 24576, False), (191, 65536, False),
    # enough of them are not
    (128, 16384, True), (140, 14976, True), (192, 65536, True), (511, 65536, True), (511, 65537, False), (512, 1 << 40, True),
])
def test_score_pass(rules, regions, values, one_pass):
    assert bool(rules.score_one_pass(regions, values, CUS)) == one_pass


def _cuts(rules, dh, heads, batch):
    """batch: (requests, active rows, tokens) groups."""
    tiles = sum(n * -(-rows // 256) for n, rows, _ in batch)
    work = sum(n * -(-rows // 256) * -(-tok // 64) for n, rows, tok in batch)
    nkv = max(-(-tok // 64) for _, _, tok in batch)
    may = rules.attn_may_cut(dh, heads, sum(n for n, _, _ in batch), sum(n * tok for n, _, tok in batch),
                             max(tok for _, _, tok in batch), CUS)
    return bool(may) and bool(rules.attn_cuts(dh, tiles, heads, work, nkv, CUS))


@pytest.mark.parametrize("batch,cut", [
    # whole items were no slower, and up to 1.5 times as fast as cut ones: few key tiles ...
    ([(8, 26, 512)], False), ([(28, 150, 512)], False), ([(16, 288, 576)], False), ([(8, 230, 768)], False),
    ([(8, 768, 768)], False), ([(28, 576, 576)], False),
    # ... whole rounds of items, or workgroups nearly all busy with one
    ([(16, 1024, 1024)], False), ([(8, 51, 1024)], False), ([(4, 1024, 1024)], False), ([(8, 2048, 2048)], False),
    ([(2, 2048, 2048)], False), ([(4, 1229, 4096)], False), ([(1, 4915, 16384)], False), ([(8, 1229, 4096)], False),
    # the largest batch: 468 items, the power limit takes the shorter share back
    ([(1, 9828, 32760)], False),
    # few long items, or a last round that is nearly empty
    ([(1, 51, 1024)], True), ([(1, 1229, 4096)], True), ([(1, 2458, 8192)], True), ([(1, 1638, 32760)], True),
    ([(1, 3276, 32760)], True), ([(1, 6552, 32760)], True), ([(1, 8192, 8192)], True), ([(2, 3072, 3072)], True),
    ([(1, 819, 16384)], True), ([(1, 16384, 16384), (2, 1024, 1024)], True),
])
def test_attention_cut_head_dim_128(rules, batch, cut):
    """12 heads of 128: the video model's."""
    assert _cuts(rules, 128, 12, batch) == cut


@pytest.mark.parametrize("batch,cut", [
    ([(8, 307, 1024)], False), ([(8, 307, 1536)], False), ([(2, 2048, 2048)], True), ([(8, 410, 2048)], True),
    ([(8, 200, 2048)], True),
])
def test_attention_cut_two_shares_per_item(rules, batch, cut):
    """8 heads of 128, 128 items on 256 workgroups (64 in the last): cut from 32 key tiles on."""
    assert _cuts(rules, 128, 8, batch) == cut


@pytest.mark.parametrize("batch,cut", [
    ([(28, 77, 512)], False), ([(16, 1024, 1024)], False), ([(28, 512, 512)], False), ([(8, 1024, 1024)], False),
    ([(2, 1536, 1536)], False), ([(4, 614, 2048)], False), ([(1, 16384, 16384)], False),
    ([(1, 51, 1024)], True), ([(1, 1024, 2048)], True), ([(8, 205, 4096)], True), ([(2, 3072, 3072)], True),
    ([(4, 1229, 4096)], True), ([(1, 9828, 32760)], True), ([(2, 512, 1024), (3, 1037, 2304), (3, 1843, 4096)], True),
])
def test_attention_cut_head_dim_64(rules, batch, cut):
    """16 heads of 64: the audio model's."""
    assert _cuts(rules, 64, 16, batch) == cut


@pytest.mark.parametrize("dh,heads,requests,tokens,may", [
    # the merge is not launched where no share of active rows would cut
    (128, 12, 1, 768, False), (128, 12, 8, 1024, False), (128, 12, 28, 1024, False), (128, 12, 48, 512, False),
    (64, 16, 16, 1024, False), (64, 16, 48, 512, False), (64, 24, 1, 768, False),
    (128, 12, 4, 1024, False), (128, 12, 16, 1536, False), (64, 16, 8, 1024, False),
    (128, 12, 1, 1024, True), (128, 12, 2, 1024, True), (128, 12, 4, 2048, True), (128, 12, 1, 32760, True), (64, 24, 1, 4096, True), (64, 16, 1, 2048, True),
])
def test_attention_may_cut(rules, dh, heads, requests, tokens, may):
    assert bool(rules.attn_may_cut(dh, heads, requests, requests * tokens, tokens, CUS)) == may


def test_attention_cut_counts_active_requests(rules):
    """One active tile of a short request beside a long skipped one: nothing to cut."""
    for dh in (64, 128):
        assert not rules.attn_cuts(dh, 1, 12, 5, 256, CUS)


def test_attention_share_bounds(rules):
    """The multiplication that stands for the division by the share count, at every argument."""
    for G in (8, 16, 24, 248, 256, 304, 512, 1000, 1024):
        inv = 0xffffffff // G + 1
        a = np.arange(G * G + 1, dtype=np.uint64)
        assert np.array_equal((a * np.uint64(inv)) >> np.uint64(32), a // np.uint64(G))


def test_attention_division(rules):
    """32-bit and larger operands, on both sides of multiples of the divisor."""
    rng = np.random.default_rng(5)
    for qb in (1, 31, 32, 33, 50, 62):
        for db in (1, 9, 31, 32, 33, 40):
            for _ in range(20):
                d = max(1, int(rng.integers(0, 1 << db)))
                q = int(rng.integers(0, 1 << qb))
                for v in (q, q // d * d, q // d * d + d - 1, max(0, q // d * d - 1)):
                    assert rules.div_steps(v, d) == v // d


def test_attention_schedule_beyond_32_bits(rules):
    """A request of 1.4 million tokens, 40 heads: more than 2^32 tile-steps."""
    n = np.array([0, 1_400_000], np.int32)
    cap = 2_000_000
    out, cut = np.zeros((cap, 8), np.int32), ctypes.c_int()
    nk, nt = -(-1_400_000 // 64), -(-1_400_000 // 256)
    k = rules.attn_pieces(64, 1, 1, *(a.ctypes.data_as(ctypes.c_void_p) for a in (n, n)), 1, 40, 256, nk,
                          out.ctypes.data_as(ctypes.c_void_p), cap, ctypes.byref(cut))
    assert nk * nt * 40 > 1 << 32 and k >= nt * 40
    steps = (out[:k, 5] - out[:k, 4]).astype(np.int64)
    assert steps.min() > 0 and steps.sum() == nk * nt * 40


@pytest.mark.parametrize("seed", range(60))
@pytest.mark.parametrize("dh", [16, 64, 128])
def test_attention_schedule_covers_every_tile_step_once(rules, seed, dh):
    """Random batches (requests without active rows, ragged ends, one token): whole and cut, walked
    and from tables, every (head, query tile) runs over all its key tiles exactly once, its pieces in
    key order in consecutive shares, each in a scratch slot of its own where the merge, which starts
    from the first, looks for it, and whole where nothing may be cut."""
    rng = np.random.default_rng([seed, dh])
    B = int(rng.choice([1, 2, 3, 17, 40]))
    H = int(rng.choice([1, 2, 12, 16]))
    G = int(rng.choice([8, 16, 64, 256, 512]))
    n = np.maximum(1, np.exp(rng.uniform(0, np.log(9000 if B < 5 else 1500), B))).astype(int)
    act = np.where(rng.random(B) < 0.2, 0, np.minimum(n, (rng.random(B) * 1.1 * n).astype(int)))
    tok = np.concatenate([[0], np.cumsum(n)]).astype(np.int32)
    cu = np.concatenate([[0], np.cumsum(act)]).astype(np.int32)
    QB = 128 if dh == 16 else 256
    nt, nk = -(-act // QB), -(-n // 64)
    want = {(h, t, b): int(nk[b]) for h in range(H) for b in range(B)
            for t in range(int(nt[:b].sum()), int(nt[:b + 1].sum()))}
    cap = len(want) + 2 * G + 8
    seen = []
    for tables in (0, 1):
        for may_cut in (0, 1):
            out, cut = np.zeros((cap, 8), np.int32), ctypes.c_int()
            k = rules.attn_pieces(dh, tables, may_cut, *(a.ctypes.data_as(ctypes.c_void_p) for a in (cu, tok)), B, H, G,
                                  int(nk.max()), out.ctypes.data_as(ctypes.c_void_p), cap, ctypes.byref(cut))
            assert 0 <= k <= cap
            items, slots = {}, set()
            for w, h, t, b, k0, k1, slot, last in out[:k].tolist():
                assert 0 <= w < G and 0 <= k0 < k1
                items.setdefault((h, t, b), []).append((k0, k1, w, slot, last))
                assert slot not in slots
                if slot >= 0:
                    assert slot < 2 * G
                    slots.add(slot)
            assert set(items) == set(want)
            for key, ps in items.items():
                ps.sort()
                x = ps[0][2]
                assert [p[2] for p in ps] == list(range(x, x + len(ps)))
                assert ps[0][0] == 0 and ps[-1][1] == want[key]
                assert all(a[1] == b_[0] for a, b_ in zip(ps, ps[1:]))
                if len(ps) == 1:
                    assert ps[0][3:] == (-1, -1)
                else:
                    assert may_cut and ps[0][4] == ps[-1][2]
                    assert [p[3] for p in ps] == [rules.attn_slot_at(x, j) for j in range(len(ps))]
            work = H * int((nt * nk).sum())
            if cut.value and work >= 4 * G:   # all shares used: share w holds [floor(w work / G), floor((w + 1) work / G))
                steps = np.zeros(G, np.int64)
                np.add.at(steps, out[:k, 0], out[:k, 5] - out[:k, 4])
                np.testing.assert_array_equal(steps, np.diff([w * work // G for w in range(G + 1)]))
            elif cut.value and work <= 4 * (G - 8):   # little work: shares of four tile-steps
                steps = np.zeros(G, np.int64)
                np.add.at(steps, out[:k, 0], out[:k, 5] - out[:k, 4])
                np.testing.assert_array_equal(steps, np.diff([min(4 * w, work) for w in range(G + 1)]))
            seen.append((tables, may_cut, cut.value, sorted(out[:k].tolist())))
    # the walked and the tabled schedule are the same
    assert [s[1:] for s in seen if s[0] == 0] == [s[1:] for s in seen if s[0] == 1]


@pytest.mark.parametrize("n_max,M,N,K,splits", [
    # the down-projections of hidden 768 and 512, few of many rows active
    (16384, 1600, 768, 3072, 3), (16384, 4864, 768, 3072, 2), (16383, 1600, 768, 3072, 3), (32760, 4864, 512, 4096, 3),
    # the last layer of hidden 3072, below 16384 rows only
    (16383, 1638, 64, 3072, 3), (32768, 1638, 64, 3072, 1),
    # wide ones split below 16384 rows only
    (8192, 512, 1536, 6144, 5), (16383, 512, 1536, 6144, 5), (16384, 512, 1536, 6144, 1), (4096, 1664, 1536, 6144, 3),
    (4096, 1664, 1536, 1536, 1),
])
def test_gemm_splits(rules, n_max, M, N, K, splits):
    assert rules.gemm_splits(n_max, M, N, K, CUS) == splits


LARGE, TALL, MID, DEEP, PAIR = range(5)


@pytest.mark.parametrize("M,N,K,shape", [
    (9728, 4608, 1536, LARGE), (8200, 3072, 1024, LARGE), (8200, 1024, 1024, TALL), (3280, 3072, 1024, TALL), (3280, 2048, 1024, MID),
    (1025, 3072, 1024, DEEP), (25, 1024, 2048, DEEP), (25, 3072, 1024, PAIR), (1025, 1024, 1024, PAIR),
    # widths of an odd number of 64 columns: more units than workgroups, so that both tiles of a pair have work
    (1280, 3264, 1088, PAIR), (2560, 3264, 1088, PAIR), (3712, 1088, 1088, PAIR), (7424, 1088, 1088, PAIR),
])
def test_large_gemm_shape(rules, M, N, K, shape):
    assert rules.large_shape(M, N, K, CUS) == shape


@pytest.mark.parametrize("M,N,K,shape", [(1664, 6144, 1536, 1), (1664, 4608, 1536, 0), (1664, 1536, 1536, 2), (4096, 6144, 1536, 0), (1664, 1536, 6144, 0)])
def test_small_gemm_shape(rules, M, N, K, shape):
    assert rules.small_shape(M, N, K, CUS) == shape


def test_gemm_kernel_lines(rules):
    assert not rules.gemm_large(8191, 1024) and rules.gemm_large(8192, 1024) and not rules.gemm_large(1 << 20, 1023)
