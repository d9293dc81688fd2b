"""Retirement in the serving loop against a stand-in batch (no GPU): a converged
job is out of its batch before the next step, whatever waits, so that a slow
job never steps beside finished ones; only rounds that the slot cap stopped
count as blocked; and the batches are empty at the end."""
import pytest

from paper_2003_01061_amd import serve
from test_serve_host import CLOCK, FakeBatch, Spec, footprint


class Watched(FakeBatch):
    """Counts the steps run with a converged job in the batch."""
    idle_particles = 0

    def step(self, k):
        Watched.idle_particles += sum(s.n for s, done in self.jobs.values() if done >= s.steps_needed)
        super().step(k)


def run(reqs, slots, pool=2_000_000):
    FakeBatch.instances.clear()
    CLOCK.t = 0.0
    Watched.idle_particles = 0
    srv = serve.Server(pool_bytes=pool, slots=slots, precision=1, chunk=20, batch_factory=Watched,
                       footprint=footprint, clock=CLOCK, sleep=CLOCK.sleep)
    res = srv.run(reqs)
    assert all(r.status == "ok" for r in res)
    assert all(not b.jobs for b in FakeBatch.instances)
    return srv, res


@pytest.mark.parametrize("dim", [2, 3])
def test_a_slow_job_does_not_step_beside_finished_ones(dim):
    reqs = [serve.Request(q, dim, 1000, 0.0, Spec(1000, 100, 20)) for q in range(6)]
    reqs.append(serve.Request(6, dim, 100, 0.0, Spec(100, 100, 2000)))
    srv, res = run(reqs, slots=8)
    assert Watched.idle_particles == 0
    # 20 steps of everything, then the slow job alone
    assert res[6].done == pytest.approx(20e-6 * 6100 + 1980e-6 * 100)


def test_free_slots_do_not_count_as_blocked():
    # as many slots as requests are ever there at once: nothing waits
    reqs = [serve.Request(q, 2 + q % 2, 500, 10.0 * q, Spec(500, 100, 40)) for q in range(6)]
    srv, _ = run(reqs, slots=1)
    assert srv.stats.blocked_slots == 0 and Watched.idle_particles == 0


def test_a_full_server_hands_slots_to_the_other_dimension():
    reqs = [serve.Request(q, 2, 500, 0.0, Spec(500, 100, 40)) for q in range(3)]
    reqs += [serve.Request(3 + q, 3, 500, 1e-6, Spec(500, 100, 40)) for q in range(3)]
    srv, res = run(reqs, slots=3)
    assert srv.stats.blocked_slots > 0 and srv.stats.max_resident <= 3
    assert min(r.admitted for r in res[3:]) >= min(r.done for r in res[:3])
    assert Watched.idle_particles == 0
