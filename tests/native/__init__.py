"""Native code that only the tests use."""
