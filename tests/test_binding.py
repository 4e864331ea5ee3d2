"""The Python binding's argument marshalling, without a GPU: the cache's buffers
are host memory and a recorder stands in for the library."""
import ctypes

import pytest
import torch

import paper_2608_28911_amd as P

B, H, D = 2, 8, 128


def make_cache(monkeypatch, **kw):
    monkeypatch.setattr(P, "_stream", lambda: 0)
    d = dict(n_layers=1, n_kv_heads=H, batch=B, base=P.BASE_AFFINE, L_hi=6, L_lo=5, group=128, r_num=26, r_den=100,
             max_prompt=2048, max_new=128)
    d.update(kw)
    return P.SemKVCache(P.make_config(**d), device="cpu")


class Recorder:
    """Every call returns 0; what its pointer arguments of `sizes` bytes hold is
    read while the call runs."""

    def __init__(self, **sizes):
        self.sizes, self.seen, self.args = sizes, {}, {}

    def __getattr__(self, name):
        def call(*args):
            self.args[name] = args
            self.seen[name] = {i: ctypes.string_at(args[i], n) for i, n in self.sizes[name].items()}
            return 0
        return call


def rows(n=64):
    """One step's K and V rows as slices of [B, H, n, 128]: not contiguous."""
    g = torch.Generator().manual_seed(3)
    K, V = (torch.randn((B, H, n, D), generator=g).half() for _ in range(2))
    k, v = K[:, :, n // 2], V[:, :, n // 2]
    assert not k.is_contiguous() and not v.is_contiguous()
    return k, v


def raw(t):
    return t.contiguous().numpy().tobytes()


def test_append_copies_of_rows_live_until_the_call(monkeypatch):
    """Rows that are not contiguous are copied: both copies are there, each with
    its own values, while the library reads their pointers."""
    n = B * H * D * 2
    c = make_cache(monkeypatch)
    c._lib = lib = Recorder(semkv_append_kv={2: n, 3: n}, semkv_append_decode={2: n, 3: n, 4: 4 * n},
                            semkv_append_commit={1: 4 * B})
    k, v = rows()
    c.append_kv(0, k, v)
    assert lib.seen["semkv_append_kv"] == {2: raw(k), 3: raw(v)}
    q = torch.randn((B, 4 * H, 2 * D)).half()[:, :, ::2]
    c.append_decode_attn(0, k, v, q, out=torch.empty((B, 4 * H, D)), workspace=torch.empty(16))
    assert lib.seen["semkv_append_decode"] == {2: raw(k), 3: raw(v), 4: raw(q)}
    s = torch.arange(2.0 * B)[::2]
    c.append_commit(s)
    assert lib.seen["semkv_append_commit"] == {1: raw(s)}


def test_calls_follow_a_replaced_struct(monkeypatch):
    """cache.c may be replaced (a saved copy of the counts, say): the library's
    calls, the counts and the list sizes are then all those of the new struct."""
    c = make_cache(monkeypatch)
    new = type(c.c).from_buffer_copy(c.c)
    new.cfg.r_num, new.n_hi, new.n_lo = 50, 100, 300
    c.c = new
    assert c.counts["n_hi"] == 100 and c.rank_sizes(200) == (100, 100)
    c._lib = lib = Recorder(semkv_rank={})
    hi, lo = c.rank(torch.zeros((B, 200)))
    assert hi.shape == (B, 100) and lo.shape == (B, 100)
    struct = lib.args["semkv_rank"][0]._obj
    assert ctypes.addressof(struct) == ctypes.addressof(new)
