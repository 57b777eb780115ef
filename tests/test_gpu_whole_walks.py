"""The tests of small shapes again, on the kernels of one walk a wave: small launches deal their walks to the waves of a
work-group and leave these kernels, which run everything large, without the edges that the tests were written for.

Whole makes of every call one with the same batch entries again and again, as many times as it takes until no launch deals its walks
(burst_attn_launch_plan), asks that all repetitions give the same bits and hands out the first.  With `apart`, dQ and dK, dV come from
a launch each, as those of large steps do."""
import pytest

from tests import (test_gpu_block_mask, test_gpu_d64_tiles, test_gpu_first_tiles, test_gpu_head_layouts, test_gpu_nonfinite,
                   test_gpu_random_descriptors, test_gpu_steps)

pytestmark = pytest.mark.gpu


class Whole:
    def __init__(self, lib, apart=False):
        self.lib, self.apart, self.calls = lib, apart, []

    def __getattr__(self, name):
        return getattr(self.lib, name)

    def _repeats(self, call, shapes, masks):
        """How often, and the launches there are then."""
        def full(s):
            m = self.lib.burst_mask_t()
            m.mode, m.q_nseg, m.k_nseg, m.pos_stride, m.q_seg_len, m.k_seg_len = self.lib.BURST_MASK_FULL, 1, 1, 1, s.sq, s.sk
            return m
        masks = [m if m is not None else full(s) for m, s in zip(masks, shapes)]
        for times in (1 << i for i in range(11)):
            more = self._shapes(shapes, times)
            try:
                kinds = self.lib.burst_attn_launch_plan(call, more, masks)
            except self.lib.BurstError:        # steps that may not share a launch
                kinds = [x for s, m in zip(more, masks) for x in self.lib.burst_attn_launch_plan(call, [s], [m])]
            if not any(x & self.lib.BURST_KERNEL_DEALT for x in kinds):
                self.calls.append(kinds)
                return times
        raise AssertionError("walks are dealt however many there are")

    def _shapes(self, shapes, times):
        return [self.lib.shape(s.batch * times, s.q_heads, s.kv_heads, s.head_dim, s.sq, s.sk, s.scale) for s in shapes]

    @staticmethod
    def _input(x, times):
        return x.expand(times, *x.shape[1:]) if x.shape[0] == 1 else x.repeat(times, *[1] * (x.dim() - 1))

    def _run(self, call, shapes, masks, inputs, outputs, fn):
        """fn(shapes, inputs, outputs) on the repeated tensors; lists of tensors stay lists, None stays None."""
        import torch
        each = lambda f, x: None if x is None else [each(f, y) for y in x] if isinstance(x, (list, tuple)) else f(x)
        times = self._repeats(call, shapes, masks)
        out = each(lambda x: x.repeat(times, *[1] * (x.dim() - 1)), outputs)
        fn(self._shapes(shapes, times), each(lambda x: self._input(x, times), inputs), out)

        def back(x, many):
            if isinstance(x, (list, tuple)):
                for a, b in zip(x, many):
                    back(a, b)
            elif x is not None and x.numel():
                same = many.view(torch.int32 if many.dtype == torch.float32 else torch.int16).reshape(times, *x.shape)
                assert bool((same == same[:1]).all())
                x.copy_(many[:x.shape[0]])
        back(outputs, out)

    def burst_attn_step_fwd(self, shp, mask, q, k, v, o_part=None, lse_part=None, o_acc=None, lse_acc=None):
        self._run("fwd" if o_part is None else "fwd_part", [shp], [mask], [q, k, v], [o_part, lse_part, o_acc, lse_acc],
                  lambda s, i, o: self.lib.burst_attn_step_fwd(s[0], mask, *i, o_part=o[0], lse_part=o[1], o_acc=o[2], lse_acc=o[3]))

    def burst_attn_steps_fwd(self, shapes, masks, q, k, v, o_acc, lse_acc):
        self._run("fwd", shapes, masks, [q, list(k), list(v)], [o_acc, lse_acc],
                  lambda s, i, o: self.lib.burst_attn_steps_fwd(s, masks, *i, *o))

    def burst_attn_step_bwd(self, shp, mask, q, k, v, d_o, lse, d, dq=None, dk=None, dv=None, accumulate_flags=0):
        def run(call, **grads):
            self._run(call, [shp], [mask], [q, k, v, d_o, lse, d], list(grads.values()),
                      lambda s, i, o: self.lib.burst_attn_step_bwd(s[0], mask, *i, **dict(zip(grads, o)), accumulate_flags=accumulate_flags))
        if dk is None:
            run("dq", dq=dq)
        elif dq is None:
            run("dkdv", dk=dk, dv=dv)
        elif self.apart:
            run("dq", dq=dq)
            run("dkdv", dk=dk, dv=dv)
        else:
            run("bwd", dq=dq, dk=dk, dv=dv)

    def burst_attn_steps_bwd(self, shapes, masks, q, k, v, d_o, lse, d, dq, dk, dv, accumulate_flags=0):
        call = "dq" if dk is None else "dkdv" if dq is None else "bwd"
        self._run(call, shapes, masks, [q, list(k), list(v), d_o, lse, d], [dq, dk, dv],
                  lambda s, i, o: self.lib.burst_attn_steps_bwd(s, masks, *i, *o, accumulate_flags=accumulate_flags))


@pytest.fixture(params=["together", "apart"])
def whole(lib, request):
    return Whole(lib, request.param == "apart")


@pytest.fixture
def whole_fwd(lib):
    return Whole(lib)


def _args(test):
    """The parametrisations of a test, to be used again."""
    def again(fn):
        for mark in test.pytestmark:
            if mark.name == "parametrize":
                fn = pytest.mark.parametrize(*mark.args, **mark.kwargs)(fn)
        return fn
    return again


@_args(test_gpu_first_tiles.test_first_key_tiles_with_scattered_rows)
def test_first_key_tiles_with_scattered_rows(whole_fwd, d, sk):
    test_gpu_first_tiles.test_first_key_tiles_with_scattered_rows(whole_fwd, d, sk)
    assert whole_fwd.calls == [[0]] * 4


@_args(test_gpu_nonfinite.test_rows_that_see_nothing_of_a_tile_are_not_touched_by_it)
def test_rows_that_see_nothing_of_a_tile_are_not_touched_by_it(whole, kind, d, blocks):
    test_gpu_nonfinite.test_rows_that_see_nothing_of_a_tile_are_not_touched_by_it(whole, kind, d, blocks)


@_args(test_gpu_head_layouts.test_short_walks)
def test_short_walks(whole, d, sk):
    test_gpu_head_layouts.test_short_walks(whole, d, sk)


@_args(test_gpu_head_layouts.test_key_tile_heights)
def test_key_tile_heights(whole, B, H, d, sq, sk, causal):
    test_gpu_head_layouts.test_key_tile_heights(whole, B, H, d, sq, sk, causal)


@_args(test_gpu_head_layouts.test_gradients_together_and_apart)
def test_gradients_together_and_apart(whole_fwd, B, Hq, Hkv, d, sq, sk, causal):
    test_gpu_head_layouts.test_gradients_together_and_apart(whole_fwd, B, Hq, Hkv, d, sq, sk, causal)


@pytest.mark.parametrize("B,Hq,Hkv,d,n,causal", [
    (1, 6, 3, 128, 2900, False),     # three keys, groups of two
    (1, 9, 9, 64, 2000, False),      # one whole round of the XCDs and one key left over
    (5, 3, 3, 64, 2400, True),       # fifteen keys over the batch
    (2, 28, 7, 128, 700, True),      # groups of four
    (2, 16, 8, 64, 1200, True),      # two whole rounds, uneven walks: the keys of an XCD side by side
])
def test_head_layouts(lib, B, Hq, Hkv, d, n, causal):
    """Not repeated: the mapping of heads to XCDs goes by their number."""
    whole = Whole(lib)
    test_gpu_head_layouts.step_case(whole, B, Hq, Hkv, d, n, n, causal, B * 1000 + Hq + n)
    mask = lib.burst_mask_t()
    mask.mode = lib.BURST_MASK_CAUSAL if causal else lib.BURST_MASK_FULL
    mask.q_nseg = mask.k_nseg = mask.pos_stride = 1
    mask.q_seg_len = mask.k_seg_len = n
    assert lib.burst_attn_launch_plan("fwd_part", [lib.shape(B, Hq, Hkv, d, n, n, 0.1)], [mask]) == [0]


@_args(test_gpu_d64_tiles.test_tiles_of_narrow_heads)
def test_tiles_of_narrow_heads(whole, sq, sk, causal):
    test_gpu_d64_tiles.test_tiles_of_narrow_heads(whole, sq, sk, causal)


@_args(test_gpu_block_mask.test_block_sparse_single_step_forward_and_backward)
def test_block_sparse_single_step(whole_fwd, d, sq, sk, bq, bk):
    test_gpu_block_mask.test_block_sparse_single_step_forward_and_backward(whole_fwd, d, sq, sk, bq, bk)


def test_all_open_block_mask_equals_no_block_mask(whole_fwd):
    test_gpu_block_mask.test_all_open_block_mask_equals_no_block_mask(whole_fwd)


def test_all_closed_block_mask(whole_fwd):
    test_gpu_block_mask.test_all_closed_block_mask(whole_fwd)


@pytest.mark.parametrize("seed", range(48))
def test_random_descriptors(lib, seed):
    test_gpu_random_descriptors.test_random_descriptor_step_against_the_oracle(Whole(lib, seed % 4 >= 2), seed)


@_args(test_gpu_steps.test_steps_in_one_call_equal_steps_one_by_one)
def test_steps_in_one_call_equal_steps_one_by_one(whole_fwd, name):
    test_gpu_steps.test_steps_in_one_call_equal_steps_one_by_one(whole_fwd, name)


@_args(test_gpu_steps.test_steps_in_one_call_are_as_exact_as_one_by_one)
def test_steps_in_one_call_are_as_exact_as_one_by_one(whole_fwd, kind, window, scales):
    test_gpu_steps.test_steps_in_one_call_are_as_exact_as_one_by_one(whole_fwd, kind, window, scales)


def test_a_nan_key_reaches_the_rows_that_see_it_in_any_step(whole_fwd):
    test_gpu_steps.test_a_nan_key_reaches_the_rows_that_see_it_in_any_step(whole_fwd)


@_args(test_gpu_steps.test_rows_that_see_nothing_in_any_step)
def test_rows_that_see_nothing_in_any_step(whole_fwd, rows, d):
    test_gpu_steps.test_rows_that_see_nothing_in_any_step(whole_fwd, rows, d)


@_args(test_gpu_steps.test_steps_that_may_not_share_a_launch_in_one_call)
def test_steps_that_may_not_share_a_launch_in_one_call(whole_fwd, what, flags):
    test_gpu_steps.test_steps_that_may_not_share_a_launch_in_one_call(whole_fwd, what, flags)


@_args(test_gpu_steps.test_infinities_in_one_call_as_in_steps_one_by_one)
def test_infinities_in_one_call_as_in_steps_one_by_one(whole_fwd, what, d):
    test_gpu_steps.test_infinities_in_one_call_as_in_steps_one_by_one(whole_fwd, what, d)
