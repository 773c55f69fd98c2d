"""The binding's two ways to the library (csrc/marshal.cpp for plain tensors, Python for the rest) take the same calls
and give the same bits: a `causal` that is no bool sends a call the Python way.  What one way refuses the other refuses."""
import ctypes
import subprocess

import pytest
import torch

from paper_2512_18134_amd import binding

pytestmark = pytest.mark.gpu


def tensors(dt, B=2, H=3, S_q=70, S_kv=130, D=64):
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    mk = lambda S: torch.empty((B, H, S, D), device="cuda").normal_(generator=g).to(dt)
    return mk(S_q), mk(S_kv), mk(S_kv), mk(S_q)


def same(a, b):
    return len(a) == len(b) and all(x.dtype == y.dtype and torch.equal(x, y) for x, y in zip(a, b))


@pytest.mark.parametrize("dt", [torch.bfloat16, torch.float16])
def test_both_ways_give_the_same(dt):
    fwd, split, bwd = ((binding.attn_fwd, binding.attn_fwd_splitkv, binding.attn_bwd) if dt == torch.bfloat16 else
                       (binding.attn_fwd_f16, binding.attn_fwd_splitkv_f16, binding.attn_bwd_f16))
    q, k, v, d_o = tensors(dt)
    assert binding._native().fwd(dt == torch.float16, q, k, v, None, None, False, None, None) is not None
    for causal in (False, True):
        o, lse = fwd(q, k, v, causal=causal)
        assert same(fwd(q, k, v, causal=int(causal)), (o, lse))
        assert o.is_contiguous() and lse.shape == q.shape[:3] and lse.dtype == torch.float32
        o2, lse2 = torch.full_like(o, 7), torch.full_like(lse, 7)
        out = fwd(q, k, v, o2, lse2, causal=causal, scale=0.25)
        assert out[0].data_ptr() == o2.data_ptr() and same(fwd(q, k, v, causal=int(causal), scale=0.25), (o2, lse2))
        grads = bwd(q, k, v, o, d_o, lse, causal=causal)
        assert same(bwd(q, k, v, o, d_o, lse, causal=int(causal)), grads)
        ws = torch.empty(2 * lse.numel(), dtype=torch.float32, device="cuda")
        given = [torch.full_like(t, 7) for t in (q, k, v)]
        assert same(bwd(q, k, v, o, d_o, lse, *given, ws, causal=causal), grads) and same(given, grads)
    part = split(q, k, v, 2)
    assert same(split(q, k, v, 2, causal=0), part)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        on_current = fwd(q, k, v)
    named = fwd(q, k, v, stream=side)
    torch.cuda.synchronize()
    assert same(on_current, fwd(q, k, v)) and same(named, on_current)
    p = torch.nn.Parameter(q)                      # gradients are not tracked, as before
    assert not fwd(p, k, v)[0].requires_grad


def test_refusals_are_the_same():
    q, k, v, d_o = tensors(torch.bfloat16)
    o, lse = binding.attn_fwd(q, k, v)
    bad_calls = [
        (TypeError, lambda c: binding.attn_fwd(q.float(), k, v, causal=c)),
        (TypeError, lambda c: binding.attn_fwd(q.transpose(1, 2), k, v, causal=c)),
        (TypeError, lambda c: binding.attn_fwd(q[0], k[0], v[0], causal=c)),
        (TypeError, lambda c: binding.attn_fwd(q.cpu(), k, v, causal=c)),
        (ValueError, lambda c: binding.attn_fwd(q, k[:, :2].contiguous(), v, causal=c)),
        (TypeError, lambda c: binding.attn_fwd(q, k, v, o=o.half(), causal=c)),
        (TypeError, lambda c: binding.attn_fwd(q, k, v, lse=lse[:, :, :1].contiguous(), causal=c)),
        (binding.AttnError, lambda c: binding.attn_fwd(q, k, v, scale=-1.0, causal=c)),
        (binding.AttnError, lambda c: binding.attn_fwd(q, k, v, scale=float("nan"), causal=c)),
        (binding.AttnError, lambda c: binding.attn_fwd(*(t[..., :32].contiguous() for t in (q, k, v)), causal=c)),
        (ValueError, lambda c: binding.attn_bwd(q, k, v, o[:, :, :5].contiguous(), d_o, lse, causal=c)),
        (TypeError, lambda c: binding.attn_bwd(q, k, v, o, d_o, lse.double(), causal=c)),
        (TypeError, lambda c: binding.attn_bwd(q, k, v, o, d_o, lse, delta_ws=lse, causal=c)),
        (binding.AttnError, lambda c: binding.attn_fwd_splitkv(q, k, v, 0, causal=c)),
        (binding.AttnError, lambda c: binding.attn_fwd_splitkv(q, k, v, 300, causal=c)),
        (binding.AttnError, lambda c: binding.attn_fwd_splitkv(q, k, v, 2, workspace=torch.empty(8, device="cuda"), causal=c)),
        (AttributeError, lambda c: binding.attn_fwd(q, k, v, stream="none", causal=c)),
    ]
    for error, call in bad_calls:
        for causal in (False, 0):
            with pytest.raises(error):
                call(causal)
    with pytest.raises(binding.AttnError):
        binding.attn_fwd_splitkv(q, k, v, 2, causal=True)


def busy(stream, x):
    """Some 20 ms of work on the stream."""
    with torch.cuda.stream(stream):
        y = torch.empty_like(x)
        for _ in range(20):
            torch.mm(x, x, out=y)
    return y


@pytest.mark.parametrize("dt", [torch.bfloat16, torch.float16])
def test_a_call_on_a_named_stream_shares_no_memory_with_the_current_one(dt):
    """What a call allocates for kernels of another stream is not given to the current stream before they have run (the
    workspaces), and is no memory that the current stream has still to write (the results)."""
    fwd, split, bwd = ((binding.attn_fwd, binding.attn_fwd_splitkv, binding.attn_bwd) if dt == torch.bfloat16 else
                       (binding.attn_fwd_f16, binding.attn_fwd_splitkv_f16, binding.attn_bwd_f16))
    q, k, v, d_o = tensors(dt, B=4, H=16, S_q=1000, S_kv=1000)
    o, lse = fwd(q, k, v)
    x = torch.ones((8192, 8192), dtype=torch.bfloat16, device="cuda")
    calls = {"fwd": lambda s: fwd(q, k, v, stream=s), "splitkv": lambda s: split(q, k, v, 3, stream=s),
             "bwd": lambda s: bwd(q, k, v, o, d_o, lse, stream=s), "fwd, not plain": lambda s: fwd(q, k, v, causal=0, stream=s)}
    sizes = [o.nbytes, lse.nbytes, 2 * lse.nbytes, binding.attn_fwd_splitkv_workspace_bytes(4, 16, 1000, 64, 3)]
    current = torch.cuda.current_stream()
    for name, call in calls.items():
        want = call(None)
        for side in (torch.cuda.Stream(), torch.cuda.ExternalStream(torch.cuda.Stream().cuda_stream)):
            print(name, dt, type(side).__name__, flush=True)
            torch.cuda.synchronize()
            keep = [busy(side, x)]
            got = call(side)                                  # waits behind the products
            keep += [torch.full((n // 4,), float("nan"), device="cuda") for n in sizes for _ in range(3)]
            torch.cuda.synchronize()
            assert same(got, want)
            del got
            keep.append(busy(current, x))
            freed = [torch.full((n // 4,), float("nan"), device="cuda") for n in sizes for _ in range(3)]
            del freed                                         # written behind the products, then free for this stream
            got = call(side)
            torch.cuda.synchronize()
            assert same(got, want)


ALLOCATOR = """
#include <sys/types.h>
int PyGILState_Check(void);
static char *slab;
static ssize_t used, size;
static int calls, locked;
void use_slab(void *p, ssize_t n) { slab = p; size = n; used = calls = locked = 0; }
void counts(int *c, int *l) { *c = calls; *l = locked; }
void *slab_alloc(ssize_t n, int device, void *stream)
{
    ++calls;
    locked += PyGILState_Check();
    n = (n + 511) / 512 * 512;
    if (used + n > size)
        return 0;
    used += n;
    return slab + used - n;
}
void slab_free(void *p, ssize_t n, int device, void *stream) {}
"""


def test_allocations_release_the_interpreter_lock(tmp_path):
    """An allocation may wait for the device: no thread is kept from running meanwhile.  Seen from a memory pool whose
    allocator asks whether the calling thread holds the lock."""
    (tmp_path / "slab.c").write_text(ALLOCATOR)
    so = str(tmp_path / "slab.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-o", so, str(tmp_path / "slab.c")], check=True)
    lib = ctypes.CDLL(so)
    memory = torch.empty(1 << 28, dtype=torch.uint8, device="cuda")
    skip = 1 << 20       # torch's allocator keys its blocks by address: none of the pool's starts where `memory` does
    lib.use_slab(ctypes.c_void_p(memory.data_ptr() + skip), ctypes.c_ssize_t(memory.nbytes - skip))
    q, k, v, d_o = tensors(torch.bfloat16, B=4, H=8, S_q=512, S_kv=512, D=128)          # every allocation more than 1 MB
    o, lse = binding.attn_fwd(q, k, v)
    allocator = torch.cuda.memory.CUDAPluggableAllocator(so, "slab_alloc", "slab_free")
    pool = torch.cuda.MemPool(allocator.allocator())
    with torch.cuda.use_mem_pool(pool):
        keep = [binding.attn_fwd(q, k, v), binding.attn_fwd_splitkv(q, k, v, 2), binding.attn_bwd(q, k, v, o, d_o, lse)]
    torch.cuda.synchronize()
    calls, locked = ctypes.c_int(), ctypes.c_int()
    lib.counts(ctypes.byref(calls), ctypes.byref(locked))
    same_o = torch.equal(keep[0][0], o)
    del keep, pool            # the pool goes before its allocator and its memory, also where an assertion fails
    assert calls.value > 0 and locked.value == 0 and same_o
