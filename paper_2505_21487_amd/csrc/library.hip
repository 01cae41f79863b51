// The library as one translation unit, hence one device code object.  The units below can be compiled each by itself,
// in 90 s side by side instead of 200, but then every one is a code object with an allocation of its own on the GPU, and
// a program that changes kernels all the time pays for it: absorbed query, decode and output projection one behind the
// other (24 sequences of 200 to 6000 tokens, two latent heads) took 142.5 to 144.2 us per round in five code objects,
// depending on their sizes, and take 142.0 in one; the decode kernel, fetched again each time, is the one that differs
// (59.1 against 58.3 us).  The decode alone, again and again, is the same.
#include "gla_decode.hip"
#include "tuned_128.hip"
#include "tuned_256.hip"
#include "tuned_512.hip"
#include "wide.hip"
