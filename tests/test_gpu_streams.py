"""What a call waits for: its own stream, and no other."""
import pytest

import pbgen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bumpy():
    return pbgen.make_problem(n=3, a=6.0, c=9.0, bump=True, t=3.0, L=1, helix=0, partials=0, kappa=0.2, seed=(9, 3),
                              center_charge=1.0)


@pytest.fixture(scope="module")
def second(bumpy):
    """GPU clock cycles of a second, the library's code objects loaded."""
    import torch

    import paper_2511_21713_amd as pb
    g = pb.Problem.from_inputs(pb.Context(0), bumpy)
    g.setup()
    g.close()
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    cycles = 10**7
    torch.cuda._sleep(cycles)
    torch.cuda.synchronize()
    a.record()
    torch.cuda._sleep(cycles)
    b.record()
    torch.cuda.synchronize()
    return int(cycles * 1000.0 / a.elapsed_time(b))


def null_stream_busy_after(call, cycles):
    import torch
    done = torch.cuda.Event()
    torch.cuda._sleep(cycles)
    done.record()
    call()
    busy = not done.query()
    torch.cuda.synchronize()
    return busy


def test_first_setup_of_a_context_leaves_the_null_stream_alone(bumpy, second):
    """The first setup of a context uploads its quadrature points on the
    stream it was given: work queued on the null stream is still running when
    it returns."""
    import paper_2511_21713_amd as pb
    g = pb.Problem.from_inputs(pb.Context(0), bumpy)
    g.set_tile_shape(8, 32)  # the same workspace for both surfaces
    assert null_stream_busy_after(g.setup, second)
    g.close()


def test_setup_grows_the_workspace_before_it_is_in_use(bumpy, second):
    """The planes of the two surfaces differ in size: the workspace is made for
    the larger at once, instead of being freed and made again between them
    (freeing device memory waits for every stream)."""
    import paper_2511_21713_amd as pb
    g = pb.Problem.from_inputs(pb.Context(0), bumpy)
    assert null_stream_busy_after(g.setup, second)
    g.close()
