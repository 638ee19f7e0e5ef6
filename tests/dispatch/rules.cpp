// Prints what the dispatch rules of the library's headers say of the calls on its standard input, one a line.
#include <stdio.h>
#include <string.h>

#include "internal.h"

int main() {
    char rule[32];
    long long rows, padded, n_req, hidden;
    while (scanf("%31s %lld %lld %lld %lld", rule, &rows, &padded, &n_req, &hidden) == 5) {
        Workspace ws;
        memset(&ws, 0, sizeof ws);
        ws.max_rows = rows;
        ws.padded = padded != 0;
        if (!strcmp(rule, "small_maps")) printf("%d\n", (int)small_maps(ws, (int32_t)n_req, (int)hidden));
        else if (!strcmp(rule, "carries_side_maps")) printf("%d\n", (int)carries_side_maps(ws, (int32_t)n_req, (int)hidden));
        else return 1;
    }
    return 0;
}
