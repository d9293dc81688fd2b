"""Retirement in the serving loop against a stand-in batch (no GPU): retired jobs
may keep their slots, but they give way to any request that needs their slot or
memory, in their own dimension and in the other, and the steps their particles
go through beside running jobs are bounded; and the batches are empty at the end."""
import pytest

from paper_2003_01061_amd import serve
from test_serve_host import CLOCK, FakeBatch, Spec, footprint


class Watched(FakeBatch):
    """Adds up the steps x particles of converged jobs in the batch."""
    idle = 0

    def step(self, k):
        Watched.idle += k * sum(s.n for s, done in self.jobs.values() if done >= s.steps_needed)
        super().step(k)


def run(reqs, slots, pool=2_000_000):
    FakeBatch.instances.clear()
    CLOCK.t = 0.0
    Watched.idle = 0
    srv = serve.Server(pool_bytes=pool, slots=slots, precision=1, chunk=20, batch_factory=Watched,
                       footprint=footprint, clock=CLOCK, sleep=CLOCK.sleep)
    res = srv.run(reqs)
    assert all(r.status == "ok" for r in res)
    assert all(not b.jobs for b in FakeBatch.instances)
    return srv, res


@pytest.mark.parametrize("limit", [0, 1_000_000])
@pytest.mark.parametrize("dim", [2, 3])
def test_what_a_slow_job_pays_for_finished_ones_is_bounded(dim, limit, monkeypatch):
    monkeypatch.setattr(serve, "PARK_LIMIT", limit)
    reqs = [serve.Request(q, dim, 1000, 0.0, Spec(1000, 100, 20)) for q in range(6)]
    reqs.append(serve.Request(6, dim, 100, 0.0, Spec(100, 100, 2000)))
    srv, res = run(reqs, slots=8)
    assert Watched.idle <= limit
    # 20 steps of everything, then the slow job and what was allowed beside it
    assert res[6].done <= 20e-6 * 6100 + 1980e-6 * 100 + 1e-6 * limit + 1e-9
    if limit == 0:
        assert res[6].done == pytest.approx(20e-6 * 6100 + 1980e-6 * 100)


def test_large_finished_jobs_leave_at_once():
    n = serve.PARK_LIMIT // 20 + 1                 # one chunk beside them is over the limit
    reqs = [serve.Request(0, 2, n, 0.0, Spec(n, 100, 20)), serve.Request(1, 2, 100, 0.0, Spec(100, 100, 400))]
    run(reqs, slots=4, pool=200_000_000)
    assert Watched.idle == 0


def test_finished_jobs_give_way_to_the_other_dimension():
    reqs = [serve.Request(q, 2, 500, 0.0, Spec(500, 100, 40)) for q in range(3)]
    reqs += [serve.Request(3 + q, 3, 500, 1.0, Spec(500, 100, 40)) for q in range(3)]
    srv, res = run(reqs, slots=3)
    # nobody ran any more when they came: admitted without a step in between
    assert all(r.admitted == pytest.approx(1.0) for r in res[3:])
    assert srv.stats.blocked_slots == 1 and srv.stats.max_resident == 3


def test_finished_jobs_give_way_to_a_request_that_needs_their_memory():
    probe, _ = run([serve.Request(0, 2, 10, 0.0, Spec(10, 10, 20))], slots=8)
    n = int(0.6 * probe.cap_particles[2])
    reqs = [serve.Request(0, 2, n, 0.0, Spec(n, 10, 40)), serve.Request(1, 2, n, 5.0, Spec(n, 10, 40))]
    srv, res = run(reqs, slots=8)
    assert res[1].admitted == pytest.approx(5.0) and srv.stats.blocked_memory == 0
