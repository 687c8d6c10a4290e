// Room for one clipping pass (host arithmetic only, no HIP).
#pragma once

#include <algorithm>
#include <cmath>

namespace rpd {

// What a clipping pass fills: piece slots, the pool of element records that outgrow their chunk's own range, the items
// of the large-capacity kernel, and the polytopes that outgrow their vertex slots.
struct PassRoom {
  long long slots = 0, records = 0, deferred = 0, big = 0;
};

constexpr long long MAX_SLOTS = 800000000;  // 2 records a slot and the pool are numbered in 31 bits
inline PassRoom within_limits(PassRoom r) {
  r.slots = std::min(r.slots, MAX_SLOTS) / 64 * 64;
  r.records = std::min(r.records, 2147483647ll - 2 * (r.slots + 64 * 16));
  r.deferred = std::min(r.deferred, 1ll << 30);
  r.big = std::min(r.big, 1ll << 20);
  return r;
}

// The first attempt at nt tets and ns sites; passes: 1 for a build, 2 for a session, whose rounds clip the tets that
// change in both states. Spheres of equal radius need most: at 0.01, 0.1, 0.33, 1 and 4 of them per tet in a cube, a tet
// has 2.4, 5.8, 10.3, 18.9 and 44 candidates and 2.0, 9.8, 25, 58 and 183 element records, of which the pool gets nearly
// all where 64 pieces have over 128 records, from 0.2 spheres per tet on (at 0.02, a tenth of them). Radii drawn from a
// wide range leave half the candidates or fewer. The room is a quarter more than that and a constant. (An uneven share
// of the sites needs less: the rules are concave in the number of sites, or linear.)
// slots12: 12 vertex slots a piece, which about 1 piece in 10^2 outgrows (16: 1 in 10^4, or 4 in 10^2 at 0.5 spheres of
// equal radius per tet); the first few of a chunk need no room.
inline PassRoom pass_room(long long nt, long long ns, int passes, bool slots12) {
  const double r = nt > 0 ? (double)ns / (double)nt : 0.0, c = std::cbrt(r * r), n = (double)nt;
  PassRoom p;
  p.slots = (long long)(passes * std::min(n * (4 + 21 * c) + 16384, 1e9));
  p.records = (long long)(passes * std::min(n * (1 + 35 * c + 35 * r) + 8192, 4e9));
  p.deferred = passes * (4 * nt + 4096);
  p.big = passes * ((passes > 1 ? 4 : 1) * (nt / (slots12 ? 32 : 256)) + (slots12 ? 4 : 1) * ns / 3 + 1024);
  return within_limits(p);
}

// After an attempt that asked for more than its room (cursors run on past their end): the rest as it was, what ran out
// by a quarter more than was asked for. False when nothing ran out or the limits leave no more. (Counts of work that an
// overflow cut short are too low; then the next attempt asks for more.)
inline bool grow(PassRoom& room, const PassRoom& asked) {
  PassRoom g = room;
  if (asked.slots > room.slots) {
    g.slots = asked.slots + asked.slots / 4 + 64;
    g.records = (long long)((double)room.records / (double)std::max(1ll, room.slots) * (double)g.slots);
  }
  if (asked.records > room.records) g.records = std::max(g.records, asked.records + asked.records / 4);
  if (asked.deferred > room.deferred) g.deferred = asked.deferred + asked.deferred / 4;
  if (asked.big > room.big) g.big = asked.big + asked.big / 4;
  g = within_limits(g);
  const bool more = g.slots > room.slots || g.records > room.records || g.deferred > room.deferred || g.big > room.big;
  room = g;
  return more;
}

}  // namespace rpd
