// Host build of the once-per-device helper: runs it for a sequence of devices and outcomes.
#include "q8_once.h"

extern "C" void q8o_run(const int *device, const int *works, int n, int *ran, int *ok)
{
    Q8OncePerDevice once;
    for (int i = 0; i < n; ++i) {
        ran[i] = 0;
        ok[i] = once(device[i], [&] { ran[i] = 1; return works[i] != 0; });
    }
}
