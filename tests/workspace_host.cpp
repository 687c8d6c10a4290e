// Test harness: the library's rule for the room of a clipping pass (workspace.h), for tests/test_workspace.py; not part
// of librpd.
#include "workspace.h"

extern "C" {
void host_pass_room(long long nt, long long ns, int passes, int slots12, long long* out) {
  const rpd::PassRoom r = rpd::pass_room(nt, ns, passes, slots12 != 0);
  out[0] = r.slots;
  out[1] = r.records;
  out[2] = r.deferred;
  out[3] = r.big;
}
int host_grow(long long* room, const long long* asked) {
  rpd::PassRoom r, a;
  r.slots = room[0], r.records = room[1], r.deferred = room[2], r.big = room[3];
  a.slots = asked[0], a.records = asked[1], a.deferred = asked[2], a.big = asked[3];
  const bool more = rpd::grow(r, a);
  room[0] = r.slots, room[1] = r.records, room[2] = r.deferred, room[3] = r.big;
  return more;
}
}
