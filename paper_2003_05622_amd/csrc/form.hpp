// Which form a dedup takes (host code; nothing here needs a GPU).
//
// All forms give the same results, so this is about time only: by size, by whether the caller lists the distinct keys
// (hps_last_unique), and by what the kernels report about the dedups before, in pinned host words that nobody waits for.
#pragma once

#include <stdint.h>

namespace hps {

// The bucket form, by what its natural buckets are; the small form (small.hpp); the plain form (sort.hpp, dedup.hpp).
constexpr int kByRange = 0, kByBorders = 1, kByHash = 2, kSmallForm = 3, kPlainForm = 4;

constexpr uint32_t kSmallMax = 1u << 16;                  // occurrences the small form takes, at most
constexpr uint64_t kBorderMaxKeys = 1u << 19;             // ... the bucket form by sampled borders
constexpr uint64_t kBucketPathMaxKeys = 12u << 20;        // ... the bucket form

// What a lookup reports about the dedup before it (table.hpp: OftenLists::report).
constexpr uint32_t kReportSlow = 2, kReportOneKey = 4, kReportMixed = 8, kReportStandIn = 16, kReportUneven = 32,
                   kReportCrowded = 64;

constexpr uint32_t kQuiet = 3;           // dedups without an hps_last_unique until a caller is taken not to want it ...
constexpr uint32_t kOftenSmall = 10, kOften = 24;      // ... if he calls it often: up to kSmallMax occurrences, beyond
constexpr uint64_t kPlainHold = 32;      // dedups in another form after one disappointed
constexpr uint64_t kHintLag = 3;         // ... after a surprise that the next lists of frequent keys will cover

struct FormChoice {
  int mode;            // 0: by size and history; 1: plain radix passes always; 2, 3, 4: bucket form whenever it can, by range, borders, hash;
                       // 5: small form up to kSmallMax, beyond by hash
  // When a dedup of the bucket form by key range had to order much of its input the slow way (frequent keys that change
  // from one mini-batch to the next), or found the keys lying unevenly in their range, the following dedups take
  // another form: for kPlainHold dedups, and twice as long each time in a row the range then disappoints again.
  uint32_t range_seen, other_seen;        // serials of the last reports acted on
  uint32_t judged;          // reports of lookups up to this one do not count: issued before the range was given up
  uint32_t strikes;
  // After such a time, one dedup goes by key range again, and the next ones only when the report on that one has
  // come: a caller who never waits may be dozens of dedups ahead of the GPU (to_probe: it is due; probe: its lookup,
  // 0: none).  Not after other causes, whose stand-ins are slower than a good key range.
  bool to_probe;
  uint32_t probe;
  uint64_t range_from;      // dedups numbered below this do not go by key range
  uint64_t n_fallbacks;     // times range_from was pushed out
  // Why, which decides what takes its place: kHotKeys, a few keys that turned frequent without warning; kSlowBuckets,
  // many frequent keys in some buckets; kUnevenKeys; kCrowdedKeys, very unevenly (next).  The plain form while the
  // stand-ins have disappointed too (dedups numbered below stand_in_from).
  enum Away { kHotKeys, kSlowBuckets, kUnevenKeys, kCrowdedKeys } away;
  uint64_t stand_in_from;
  // After a mini-batch that did not suit the small form (small.hpp), the next ones that would take it go by hash: for kPlainHold
  // dedups, and twice as long each time the small form disappoints again before as many have gone well.  Then one dedup tries it,
  // and the next ones wait for what comes of that, as above.
  uint32_t small_seen;      // serial (of the dedup) of the last report acted on
  uint32_t small_judged;    // reports of dedups up to this one do not count: issued before the form was given up
  uint32_t small_strikes;
  bool small_doubted;       // it has disappointed, and no try since then has gone well
  uint32_t small_try;       // the lookup of the dedup that tries it, 0: none
  uint64_t small_from;      // dedups numbered below this do not take the small form
  uint32_t unlisted;        // dedups of pulls since the last hps_last_unique (or the creation)
  // ... and how many there were the time before.  Keys dealt out by hash have to be sorted when they are listed, which costs as much as
  // so many mini-batches by hash gain (often).  Whoever has just listed after no more than that keeps an order of keys for as many
  // dedups again, so that a caller with such a period is caught once; whoever lists more rarely is better off by hash all the same.
  // (us a step, hashed keys, dim 16, by range always and by hash from the fourth dedup after a listing on, a listing every
  // 4, 12, 48 steps: 1000 occurrences 38, 37, 36 and 59, 37, 29; 20 K 49, 47, 46 and 73, 42, 30; 0.3 M 81, 77, 76 and 112, 83, 73;
  // 2 M 297, 287, 283 and 358, 302, 281; 9 M 1314, 1283, 1271 and 1500, 1316, 1246.  The two meet at 13, 9, 23, 34 and 20.)
  uint32_t period;
  static uint32_t often(uint64_t n) { return n <= kSmallMax ? kOftenSmall : kOften; }
  uint32_t patience(uint64_t n) const { return period && period <= often(n) ? often(n) : kQuiet; }
  // hps_last_unique is called for a mini-batch for the first time.
  void listed() {
    period = unlisted ? unlisted : 1;       // (0: a dedup may have come before the listing of the one before it)
    unlisted = 0;
  }
  // Since an hps_last_unique was captured: the form, plus 1, of the mini-batch it was captured for.  A replay lists a later
  // mini-batch of as many occurrences with the kernels of that form, so all of these have to take it, whatever is
  // reported and listed.  By sizes that have the same forms to choose from (pin_of), 0: none.
  uint8_t pinned[3];
  // The same for the plain form itself: after a dedup whose keys agreed in all the bits the
  // plain form sorts by (kReportMixed), the following ones sort by all 64 bits.
  uint32_t full_strikes;
  uint64_t full_until;
  uint64_t n_full_fallbacks;

  // The words the lookups report into: of dedups by key range, of dedups in any other form; and the one of the small form.
  struct Reports {
    unsigned long long range, other, small;
  };

  static int pin_of(uint64_t n) { return n <= kSmallMax ? 0 : n <= kBorderMaxKeys ? 1 : n <= kBucketPathMaxKeys ? 2 : -1; }
  // hps_last_unique is captured for a mini-batch of n occurrences that was dealt out in this form.
  void captured(uint64_t n, int form) {
    const int p = pin_of(n);            // (beyond there is the plain form only)
    if (p >= 0 && !pinned[p]) pinned[p] = (uint8_t)(form + 1);
  }

  // The form of dedup number `serial`, of n occurrences, with lookup_serial lookups issued so far.  listable: of a
  // mini-batch whose distinct keys may be listed (a pull's).
  int next(uint32_t n, bool listable, uint64_t serial, uint64_t lookup_serial, Reports reports) {
    // The bucket path needs to know the heavy keys, which it learns from the lookups: the
    // first two dedups of a table take the plain passes, as do very large ones.
    const bool small = n <= kBorderMaxKeys, lists = unlisted < 2;       // (the next dedup may come before the call)
    const bool quiet = !listable || unlisted >= patience(n);
    if (listable && unlisted < ~0u) ++unlisted;
    if (mode == 0) take(reports, serial, lookup_serial, small, lists);
    const int pin = pin_of(n);
    if (mode == 0 && listable && pin >= 0 && pinned[pin]) return pinned[pin] - 1;
    // The stand-ins for the key range.  By hash is the fastest for uneven keys whatever the size, but hps_last_unique then
    // has to sort all distinct keys.  So a caller who lists the keys of his mini-batches keeps an order of keys: up to
    // kBorderMaxKeys by range as long as that is not several times slower, else by borders; above, the plain form.
    // By borders also where frequent keys, not uneven ones, made buckets slow.
    // (Raw ids, a tenth of the occurrences in a 200th of their range, a step at dim 16 of 105 K, 300 K, 1 M and 4 M occurrences:
    // by range 327, 402, 1494 and 5822 us, by hash 76, 104, 263 and 940, plain 126, 187, 391 and 1270, by borders 118 and 161; ids whose
    // density rises from none to twice the mean: by range 90, 125, 740 and 2057, by hash 76, 104, 279 and 900.
    // Listing the unique keys: 18 to 40 us by borders, in the plain form 5 to 20, by hash 620 for 4 M distinct keys.)
    if (n <= kSmallMax && (mode == 5 || (mode == 0 && quiet && small_suits(serial, lookup_serial)))) return kSmallForm;
    if (n > kBucketPathMaxKeys || mode == 1 || (mode == 0 && lookup_serial < 2)) return kPlainForm;
    if (mode != 0) return mode == 3 && small ? kByBorders : mode >= 4 ? kByHash : kByRange;
    // (Nobody wants the keys in order: by hash.  The first kernel has no key range to sample, and a bucket's rows lie in one
    // part of the table.  Hashed keys, dim 16, four steps of 2 M and 9.8 M occurrences: by range 1104 and 4787 us, by hash 1080 and
    // 4735; 0.3 M accumulated, 77 and 73.  With hps_last_unique it is the other way round: above.)
    if (quiet) return serial >= stand_in_from ? kByHash : kPlainForm;
    if (serial >= range_from && !probe) {
      if (to_probe) {
        probe = (uint32_t)lookup_serial + 1;
        to_probe = false;
      }
      return kByRange;
    }
    if (away == kUnevenKeys && lists && small) return kByRange;
    const int form = away >= kUnevenKeys && !lists ? kByHash : kByBorders;
    return away != kHotKeys && (small || form == kByHash) && serial >= stand_in_from ? form : kPlainForm;
  }

  // Whether a plain dedup sorts by all 64 bits of the keys.
  bool all_bits(uint64_t serial) const { return mode < 2 && serial < full_until; }

 private:
  bool small_suits(uint64_t serial, uint64_t lookup_serial) {
    if (serial < small_from || small_try) return false;
    if (small_doubted) small_try = (uint32_t)lookup_serial + 1;
    return true;
  }

  void take(Reports reports, uint64_t serial, uint64_t lookup_serial, bool small, bool lists) {
    if ((uint32_t)reports.range != range_seen) {
      const uint32_t at = (uint32_t)reports.range, flags = (uint32_t)(reports.range >> 32);
      range_seen = at;
      if (probe && (int32_t)(at - probe) >= 0) probe = 0;
      const bool uneven = (flags & kReportUneven) && !(lists && small && !(flags & kReportCrowded));
      if ((int32_t)(at - judged) <= 0) {
        // (of a dedup that was under way when the range was given up)
      } else if (uneven || (flags & kReportSlow)) {
        ++n_fallbacks;
        judged = (uint32_t)lookup_serial;
        if (uneven) {
          away = (flags & kReportCrowded) ? kCrowdedKeys : kUnevenKeys;
        } else {
          // (a few keys that turned frequent: plain until the hint has caught up)
          away = (flags & kReportOneKey) ? kHotKeys : kSlowBuckets;
        }
        to_probe = uneven;
        if (away == kHotKeys) {
          range_from = serial + kHintLag;
        } else {
          range_from = serial + (kPlainHold << (strikes < 7 ? strikes : 7));
          ++strikes;
        }
      } else {
        strikes = 0;
      }
    }
    if ((uint32_t)reports.small != small_seen) {
      const uint32_t at = small_seen = (uint32_t)reports.small;
      if ((int32_t)(at - small_judged) > 0) {
        if (!small_doubted && (int32_t)(at - (uint32_t)small_from) > (int32_t)kPlainHold) small_strikes = 0;
        small_judged = (uint32_t)serial - 1;
        small_doubted = true;
        small_try = 0;
        small_from = serial + (kPlainHold << (small_strikes < 7 ? small_strikes : 7));
        ++small_strikes;
      }
    }
    if ((uint32_t)reports.other != other_seen) {
      const uint32_t at = (uint32_t)reports.other, flags = (uint32_t)(reports.other >> 32);
      other_seen = at;
      // (of a lookup after the try's: what that had to report would be here)
      if (small_try && (int32_t)(at - small_try) > 0) {
        small_try = 0;
        small_doubted = false;
      }
      if (probe && (int32_t)(at - probe) >= 0) {      // its dedup was replaced by another: try again
        probe = 0;
        to_probe = true;
      }
      if ((flags & kReportStandIn) && (flags & kReportSlow)) {
        stand_in_from = serial + ((flags & kReportOneKey) ? kHintLag : kPlainHold);
      }
      if (flags & kReportMixed) {
        // the plain form's sorted bits did not tell the keys apart: all 64 bits for a while
        full_until = serial + (kPlainHold << (full_strikes < 7 ? full_strikes : 7));
        ++full_strikes;
        ++n_full_fallbacks;
      } else if (!(flags & kReportStandIn) && serial >= full_until) {
        full_strikes = 0;       // the plain form with its usual passes did well
      }
    }
  }
};

}  // namespace hps
