// The count of workgroups that leave a launch whose counters calls without a plan share (last_to_leave), with memory that lets other
// workgroups act between any two accesses of one: after launches that overlapped, the count is 0, and somebody has cleared what they left
// behind after the last of them was done.
#include <cstdio>
#include <cstdlib>

#include "flexsp_internal.h"

struct Chip {
    unsigned left = 0, grid, seed;
    int waiting;     // workgroups that have not left yet
    int inside = 0;  // workgroups that are leaving
    long tickets = 0;

    unsigned random(unsigned n) { return (seed = seed * 1664525u + 1013904223u) / 65536u % n; }
    void others()  // whoever comes between two accesses
    {
        while (inside < 200 && waiting > 0 && random(3) == 0) leave();
    }
    struct Left {
        Chip &chip;
        unsigned add(unsigned n)
        {
            chip.others();
            const unsigned before = chip.left;
            chip.left += n;
            chip.others();
            return before;
        }
    };
    void leave()
    {
        waiting--;
        inside++;
        tickets += random(4);  // (what it drew is there before it leaves)
        if (flexsp::last_to_leave(Left{*this}, grid)) {
            others();
            tickets = 0;
        }
        inside--;
    }
};

int main()
{
    for (unsigned seed = 1; seed <= 20000; seed++) {
        Chip c;
        c.seed = seed;
        c.grid = 1 + c.random(9);
        const int launches = 1 + (int)c.random(4);
        for (int round = 0; round < 2; round++) {
            c.waiting = launches * (int)c.grid;
            while (c.waiting > 0) c.leave();
            if (c.left != 0 || c.tickets != 0) {
                std::fprintf(stderr, "FAILED: seed %u, %d launches of %u: %u left, %ld tickets\n", seed, launches, c.grid, c.left, c.tickets);
                return 1;
            }
        }
    }
    std::printf("ok\n");
    return 0;
}
