// Host-side check of the slot-table pass's key list (tlmpm_keys.h): every sequence of eight
// additions over six keys and "no key" (~0), against the set of the keys added.  A list of
// up to four distinct keys must hold them, ascending, without asking for the longer list;
// a fifth must ask for it.
// Prints "sequences <n> four <f> wrong <w>": f sequences of exactly four distinct keys.
// Runs on the CPU only (no HIP runtime call).
#include <stdint.h>
#include <stdio.h>

#include "../../paper_2609_27342_amd/csrc/tlmpm_keys.h"

int main()
{
    const uint32_t key[7] = {~0u, 0u, 1u, 5u, 0x8000u, 0x10001u, 0x3FFFFFFFu}; // ascending from the second on
    long long n = 0, four = 0, wrong = 0;
    for (int code = 0; code < 7 * 7 * 7 * 7 * 7 * 7 * 7 * 7; code++) {
        FourKeys k;
        unsigned seen = 0;
        for (int i = 0, c = code; i < 8; i++, c /= 7) {
            k.add(key[c % 7]);
            if (c % 7) seen |= 1u << (c % 7);
        }
        const int distinct = __builtin_popcount(seen);
        n++;
        four += distinct == 4;
        bool ok = k.more == (distinct > 4);
        if (distinct <= 4) {
            ok = ok && k.count() == distinct;
            int at = 0;
            for (int j = 1; j < 7; j++)
                if (seen >> j & 1) ok = ok && k.a[at++] == key[j];
            for (; at < 4; at++) ok = ok && k.a[at] == ~0u;
        }
        wrong += !ok;
    }
    printf("sequences %lld four %lld wrong %lld\n", n, four, wrong);
    return wrong ? 1 : 0;
}
