"""Which form a call takes (host decisions only, so this runs without a GPU): the lines of the dispatch rules, and that no rule asks for
more scratch than the call has."""
import ctypes as C

from paper_2408_04275_amd import binding as mm


# the memory-side cache holds 256 MB; a shard whose arrays may still lie there from the pass before is not streamed
def test_optimizer_streams_only_what_cannot_be_cached():
    route = mm.load_library().mmtrain_route_adam
    route.argtypes = [C.c_int64, C.c_int32]
    for n, param_bytes, streamed in [(4 << 20, 2, 0), (12 << 20, 2, 0), (16 << 20, 2, 0), ((20 << 20) - 1, 2, 0), (20 << 20, 2, 1),
                                     (18 << 20, 4, 1), (17 << 20, 4, 0), (20 << 20, 0, 0), (24 << 20, 0, 1), (1 << 30, 2, 1)]:
        assert route(n, param_bytes) == streamed, (n, param_bytes)
