"""CPU: Server.close beside a thread in Server.wait, with a stand-in for the
library: nothing of the server is entered once it is destroyed, and the waiter
leaves with an error."""
from __future__ import annotations

import threading
import time

import pytest

import paper_2404_01817_amd as neat


class FakeLib:
    """A server whose requests never end; wait sleeps for its timeout."""

    def __init__(self):
        self.inside = 0
        self.after_destroy = []
        self.inside_at_destroy = None
        self.destroyed = False

    def neat_server_create(self, cfg, out):
        out._obj.value = 1234
        return 0

    def neat_server_destroy(self, h):
        self.inside_at_destroy = self.inside
        self.destroyed = True
        return 0

    def _enter(self, name):
        if self.destroyed:
            self.after_destroy.append(name)

    def neat_poll(self, h, ticket, res):
        self._enter("poll")
        return 1

    def neat_wait(self, h, ticket, timeout_us, res):
        self._enter("wait")
        self.inside += 1
        time.sleep(timeout_us * 1e-6)
        self.inside -= 1
        return 1

    def neat_last_error(self):
        return b"from the stand-in"


@pytest.mark.parametrize("waiters", [1, 3])
def test_close_waits_for_waiters(monkeypatch, waiters):
    fake = FakeLib()
    monkeypatch.setattr(neat, "lib", lambda: fake)
    server = neat.Server()
    errors = []

    def wait():
        try:
            server.wait(7, timeout_s=30.0)
        except neat.NeatError as e:
            errors.append(e.code)

    th = [threading.Thread(target=wait) for _ in range(waiters)]
    for t in th:
        t.start()
    time.sleep(0.1)  # each of them inside the library
    assert fake.inside == waiters
    t0 = time.monotonic()
    server.close()
    for t in th:
        t.join(5.0)
    assert time.monotonic() - t0 < 5.0  # not the waiters' 30 s
    assert fake.inside_at_destroy == 0 and fake.after_destroy == []
    assert errors == [neat.NEAT_E_SHUTDOWN] * waiters
    server.close()  # again: nothing


def test_close_in_a_signal_handler_of_the_waiter(monkeypatch):
    import signal
    fake = FakeLib()
    monkeypatch.setattr(neat, "lib", lambda: fake)
    server = neat.Server()
    old = signal.signal(signal.SIGALRM, lambda *a: server.close())
    try:
        signal.setitimer(signal.ITIMER_REAL, 0.06)
        with pytest.raises(neat.NeatError):
            server.wait(7, timeout_s=30.0)
    finally:
        signal.signal(signal.SIGALRM, old)
    assert fake.destroyed and fake.after_destroy == []


def test_wait_times_out(monkeypatch):
    monkeypatch.setattr(neat, "lib", lambda fake=FakeLib(): fake)
    server = neat.Server()
    with pytest.raises(TimeoutError):
        server.wait(7, timeout_s=0.01)


def test_close_waits_for_a_first_look(monkeypatch):
    """A thread on its way through wait's first look at the ticket counts too."""
    fake = FakeLib()
    sleeping = fake.neat_wait
    fake.neat_wait = lambda h, ticket, us, res: sleeping(h, ticket, max(us, 200000), res)
    monkeypatch.setattr(neat, "lib", lambda: fake)
    server = neat.Server()
    errors = []

    def wait():
        try:
            server.wait(7, timeout_s=30.0)
        except neat.NeatError as e:
            errors.append(e.code)

    t = threading.Thread(target=wait)
    t.start()
    while fake.inside == 0:
        time.sleep(0.001)
    server.close()
    t.join(5.0)
    assert fake.inside_at_destroy == 0 and fake.after_destroy == []
    assert errors == [neat.NEAT_E_SHUTDOWN]
