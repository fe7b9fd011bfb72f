// Books of the turns without a device: the word that kernels write is a
// variable here, set when a launch is to have ended.
#include <cstdio>
#include <cstdlib>

#include "rdos_turn.h"

using namespace rdos;

static int failures = 0;
static void expect(bool ok, const char *what)
{
    std::printf("%s: %s\n", ok ? "ok" : "FAILED", what);
    failures += !ok;
}

int main()
{
    const int x = 0, y = 0;
    const void *caller = &x, *other = &y;
    StreamOwners owners;
    {
        LaunchTurn turn;
        uint64_t word = 0;
        const uint64_t a = owners.own_stream(), b = owners.own_stream();
        expect(a != b, "own streams are owners of their own");
        expect(turn.take(a, word, 10) == 1 && turn.take(a, word, 10) == 2, "an owner's launches follow one another");
        expect(turn.take(b, word, 10) == 0, "another owner is refused while they run");
        word = 1;
        expect(turn.take(b, word, 10) == 0, "and while the last of them runs");
        word = 2;
        expect(turn.take(b, word, 10) == 3, "and has its turn when the last has ended");
        expect(turn.take(a, word, 10) == 0, "then the first is refused");
        turn.give_back();
        expect(turn.take(a, word, 10) == 3, "a launch that the runtime refused holds nobody up");
        word = 3;
        // the stream of a is destroyed: nothing of it is asked again
        expect(turn.take(b, word, 10) == 4, "the turn goes on without the last owner's stream");
    }
    {
        LaunchTurn turn;
        const uint64_t a = owners.join(caller), b = owners.join(caller), c = owners.join(other);
        expect(a == b && a != c, "simulations on one stream are one owner");
        expect(turn.take(a, 0, 10) == 1 && turn.take(b, 0, 10) == 2 && turn.take(c, 0, 10) == 0, "and launch behind each other");
        owners.leave(caller);
        expect(owners.join(caller) == a, "as long as one of them is on it");
        owners.leave(caller);
        owners.leave(caller);
        const uint64_t d = owners.join(caller);
        expect(d != a && d != c, "a stream made later at the same address is another owner");
        expect(turn.take(d, 1, 10) == 0 && turn.take(d, 2, 10) == 3, "which waits for the first one's launches");
        owners.leave(&owners);
        expect(owners.join(other) == c, "a stream that never joined leaves nothing behind");
    }
    {
        LaunchTurn turn;
        expect(turn.take(1, 0, 100) == 1 && turn.take(2, 0, 100) == 0, "a run of 100 periods is under way");
        expect(turn.worth_waiting(0, 0, 50) && !turn.worth_waiting(0, 0, 49), "50 periods wait for it, 49 do not");
        expect(turn.take_behind(2, 50) == 2, "the second run waits");
        expect(!turn.worth_waiting(0, 0, 74) && turn.worth_waiting(0, 0, 75), "150 periods under way");
        expect(turn.worth_waiting(0, 1, 25) && !turn.worth_waiting(0, 1, 24), "50 of them after the first owner's own");
        expect(turn.worth_waiting(1, 0, 25) && !turn.worth_waiting(1, 0, 24), "or once the first run has ended");
        expect(turn.take(1, 1, 25) == 0 && turn.take_behind(1, 25) == 3, "the first owner waits in its turn");
        expect(turn.take(3, 2, 1) == 0 && turn.take(3, 3, 1) == 4, "and the turn is free when the last run has ended");
        turn.give_back();
        expect(turn.worth_waiting(2, 0, 13) && !turn.worth_waiting(2, 0, 12), "a refused launch does not count");
        for (int i = 0; i < 300; ++i) turn.take_behind(1, 0);
        expect(!turn.worth_waiting(3, 0, 1000) && turn.worth_waiting(300, 0, 0), "more launches than the books keep");
    }
    return failures ? EXIT_FAILURE : EXIT_SUCCESS;
}
