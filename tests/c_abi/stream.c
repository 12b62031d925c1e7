/* Steady traffic for a test: n short collectives (ids 0 .. n-1) that are submitted on all ranks again as soon as the oldest of them is complete,
   and the collective with id n submitted into it once.  In C: the daemon is faster than an interpreter's loop.  gcc -shared. */
#include "dfx.h"

/* sends, recvs: per id 0 .. n, nranks pointers.  Returns how many short ones were completed from the submission of id n until it was seen complete
   (looked at every 16), 0 if it was not within `most`, or a negative status.  Leaves with everything complete. */
long stream_turn(dfx_ctx* ctx, int nranks, int n, const void** sends, void** recvs, long ahead, long most) {
  const uint64_t s = 1000000000ull;
  long k, seen = 0;
  int i, r, rc = 0;
  for (i = 0; i < n && !rc; ++i) rc = dfx_submit_all(ctx, i, sends + (long)i * nranks, recvs + (long)i * nranks, 5 * s);
  for (k = 0; k < ahead + most && !rc && !seen; ++k) {
    i = (int)(k % n);
    for (r = 0; r < nranks && !rc; ++r) rc = dfx_wait(ctx, r, i, 5 * s);
    if (!rc) rc = dfx_submit_all(ctx, i, sends + (long)i * nranks, recvs + (long)i * nranks, 5 * s);
    if (!rc && k == ahead) rc = dfx_submit_all(ctx, n, sends + (long)n * nranks, recvs + (long)n * nranks, 5 * s);
    if (!rc && k > ahead && (k - ahead) % 16 == 0) {
      seen = k - ahead;
      for (r = 0; r < nranks; ++r) if (dfx_wait(ctx, r, n, 0) != DFX_OK) seen = 0;
    }
  }
  if (!rc) rc = dfx_wait_all(ctx, 10 * s);
  return rc ? rc : seen;
}
